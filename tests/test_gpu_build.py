"""GPU parity of the database-side entry points: list layouts (Fig. 2), inverted-index build (Section 2.2)."""

import numpy as np
import pytest

from gpu_common import to_gpu, idx_np
from test_gpu_ivf import build_ivf

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    import torch
    assert torch.cuda.is_available()
    import paper_1704_07355_amd as Q
    Q.lib()
    return Q


@pytest.fixture(scope="module")
def O():
    from oracle import qadc_oracle as O
    return O


# ------------------------------------------------------------------ layouts

@pytest.mark.parametrize("m", [8, 16, 32, 64])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 37, 511, 4096, 100_003])
def test_pack_and_unpack_match_oracle(Q, O, m, n):
    rng = np.random.default_rng(m * 1000 + n)
    codes = rng.integers(0, 256, size=(n, m // 2), dtype=np.uint8)
    want = O.pack_transposed(codes)
    assert Q.qadc_packed_bytes(n, m, Q.QADC_LAYOUT_TRANSPOSED) == len(want) == O.transposed_bytes(n, m)
    assert Q.qadc_packed_bytes(n, m, Q.QADC_LAYOUT_STANDARD) == codes.size
    g = to_gpu(codes)
    packed = Q.qadc_pack_codes(g, Q.QADC_LAYOUT_TRANSPOSED)
    assert np.array_equal(packed.cpu().numpy(), want)          # byte for byte, zero fill included
    import torch
    back = torch.full((n, m // 2), 0xEE, dtype=torch.uint8, device="cuda:0")
    Q.qadc_unpack_codes(packed, n, m, Q.QADC_LAYOUT_TRANSPOSED, out=back)
    assert np.array_equal(back.cpu().numpy(), codes)
    same = Q.qadc_pack_codes(g, Q.QADC_LAYOUT_STANDARD)
    assert np.array_equal(same.cpu().numpy().reshape(n, m // 2), codes)


def test_unpack_does_not_write_past_the_list(Q, O):
    import torch
    n, m = 37, 8   # 37 * 4 = 148 bytes: the list ends inside a 16-byte piece
    rng = np.random.default_rng(2)
    codes = rng.integers(0, 256, size=(n, m // 2), dtype=np.uint8)
    packed = to_gpu(O.pack_transposed(codes))
    buf = torch.full((n + 16, m // 2), 0xEE, dtype=torch.uint8, device="cuda:0")
    Q.qadc_unpack_codes(packed, n, m, Q.QADC_LAYOUT_TRANSPOSED, out=buf[:n])
    got = buf.cpu().numpy()
    assert np.array_equal(got[:n], codes) and (got[n:] == 0xEE).all()


def test_scan_of_an_unpacked_list_equals_block_scan(Q, O):
    """A database kept in the paper's transposed layout: unpack on the GPU, scan, compare with Alg. 2
    run by the oracle over the blocks and rows of the transposed list."""
    rng = np.random.default_rng(9)
    n, m, R = 20_011, 16, 50
    codes = rng.integers(0, 256, size=(n, m // 2), dtype=np.uint8)
    packed = O.pack_transposed(codes)
    qlut = rng.integers(0, 40, size=(1, m, 16), dtype=np.uint8)
    sums = O.scan_blocks_transposed(qlut[0], packed, n)
    wi, wd = O.top_r(sums, R)
    std = Q.qadc_unpack_codes(to_gpu(packed), n, m, Q.QADC_LAYOUT_TRANSPOSED)
    idx, dist = Q.qadc_scan_topk(Q.QADC_U8_4BIT, std, to_gpu(qlut), R)
    assert np.array_equal(idx_np(idx)[0], wi) and np.array_equal(dist.cpu().numpy()[0], wd)


def test_layout_errors(Q):
    import torch
    g = torch.zeros((64, 8), dtype=torch.uint8, device="cuda:0")
    out = torch.zeros((1024,), dtype=torch.uint8, device="cuda:0")
    L = Q.lib()
    import ctypes
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    assert L.qadc_pack_codes(p(g), 64, 16, 7, p(out), None) == Q.QADC_EINVAL          # unknown layout
    assert L.qadc_pack_codes(p(g), 64, 12, 1, p(out), None) == Q.QADC_EINVAL          # unsupported m
    assert L.qadc_pack_codes(p(g), -1, 16, 1, p(out), None) == Q.QADC_EINVAL
    assert L.qadc_pack_codes(p(g), 64, 16, 1, p(g), None) == Q.QADC_EINVAL            # in place
    assert L.qadc_pack_codes(p(g), 64, 16, 1, ctypes.c_void_p(out.data_ptr() + 4), None) == Q.QADC_EINVAL
    assert L.qadc_pack_codes(None, 64, 16, 1, p(out), None) == Q.QADC_EINVAL
    assert L.qadc_pack_codes(None, 0, 16, 1, None, None) == Q.QADC_OK                 # nothing to do
    assert Q.qadc_packed_bytes(10, 12, 1) == 0 and Q.qadc_packed_bytes(10, 16, 5) == 0


# ------------------------------------------------------------------ encode

@pytest.mark.parametrize("shape", [(128, 16, 16), (128, 32, 16), (96, 8, 256), (96, 16, 16), (960, 32, 16)])
def test_pq_encode_is_bit_exact(Q, O, shape):
    from oracle import cref
    d, m, k = shape
    rng = np.random.default_rng(d + m)
    n = 6007
    cb = rng.uniform(0, 255, size=(m, k, d // m)).astype(np.float32)
    x = rng.uniform(0, 255, size=(n, d)).astype(np.float32)
    x[:k] = np.concatenate([cb[j] for j in range(m)], axis=1)[:k]     # vectors that sit on centroids
    cb[:, 3] = cb[:, 1]                                                # a duplicated centroid: ties
    want = cref.pq_encode(x, cb)
    got = Q.qadc_pq_encode(to_gpu(cb), to_gpu(x)).cpu().numpy()
    assert np.array_equal(got, want)


# ------------------------------------------------------------------ inverted index

@pytest.mark.parametrize("K,d,n", [(300, 128, 5003), (64, 20, 1000), (1, 32, 100), (1000, 96, 2049)])
def test_ivf_assign_matches_oracle(Q, O, K, d, n):
    rng = np.random.default_rng(K + d)
    coarse = rng.uniform(0, 255, size=(K, d)).astype(np.float32)
    if K > 10:
        coarse[7] = coarse[2]        # duplicate centroids: the lower cell must win
        coarse[K - 1] = coarse[5]
    x = rng.uniform(0, 255, size=(n, d)).astype(np.float32)
    x[:min(n, K)] = coarse[:min(n, K)]   # vectors that sit on centroids (distance zero)
    x[-1] = coarse[K - 1]
    want = O.ivf_assign(x, coarse)
    got = Q.qadc_ivf_assign(to_gpu(coarse), to_gpu(x)).cpu().numpy()
    assert got.dtype == np.int32 and np.array_equal(got, want)
    if K > 10:
        assert got[7] == 2 and got[-1] == 5


def _closest(x, coarse):
    """Closest cell by float64 differences, lowest cell among equals; x in pieces that fit the memory."""
    x, c = np.asarray(x, np.float64), np.asarray(coarse, np.float64)
    step = max(1, 4_000_000 // c.size)
    return np.concatenate([((x[i:i + step, None] - c[None]) ** 2).sum(2).argmin(1) for i in range(0, len(x), step)])


# every width of the matrix filter (and one beyond it), tails of tiles of cells and of vectors, both vector tiles
@pytest.mark.parametrize("d,K,n", [(7, 5, 1), (32, 33, 127), (33, 64, 129), (64, 65, 300), (65, 31, 257), (96, 97, 128),
                                   (100, 200, 385), (128, 1000, 640), (129, 40, 130), (252, 300, 129), (256, 32, 200),
                                   (257, 20, 129), (16, 3, 131_073), (64, 70, 131_200), (90, 33, 131_072),
                                   (128, 65, 131_111)])
@pytest.mark.parametrize("kind", ["uniform", "offset", "ties"])
def test_ivf_assign_exact_on_close_calls(Q, d, K, n, kind):
    """The matrix filter may not decide a close call: far from the origin its margin spans many cells, and with
    small whole components many cells are exactly equally close (their squared differences are exact in float64, so
    the order of the reference's sums does not matter)."""
    rng = np.random.default_rng(d * K + n)
    if kind == "ties":
        coarse = rng.integers(0, 3, size=(K, d)).astype(np.float32)
        x = rng.integers(0, 3, size=(n, d)).astype(np.float32)
    else:
        base = 3000.0 if kind == "offset" else 0.0
        coarse = (base + rng.uniform(0, 1, size=(K, d))).astype(np.float32)
        x = (base + rng.uniform(0, 1, size=(n, d))).astype(np.float32)
        x[:min(n, K)] = coarse[:min(n, K)]
    got = Q.qadc_ivf_assign(to_gpu(coarse), to_gpu(x)).cpu().numpy()
    assert np.array_equal(got, _closest(x, coarse))


def test_ivf_assign_values_at_the_ends_of_float32(Q):
    """Squares beyond float32, below it, infinities and NaN: the float64 distances decide, an infinite distance
    loses to a finite one, the lowest cell wins among infinite ones, and a vector with a NaN keeps its marker."""
    rng = np.random.default_rng(3)
    for scale in (1e25, 1e-18, 1e-30):
        coarse = (scale * rng.uniform(0, 1, size=(70, 24))).astype(np.float32)
        x = (scale * rng.uniform(0, 1, size=(150, 24))).astype(np.float32)
        assert np.array_equal(Q.qadc_ivf_assign(to_gpu(coarse), to_gpu(x)).cpu().numpy(), _closest(x, coarse)), scale
    coarse = rng.uniform(0, 1, size=(70, 24)).astype(np.float32)
    x = rng.uniform(0, 1, size=(150, 24)).astype(np.float32)
    want = _closest(x, coarse)
    x[3, 5], x[149, 0] = np.inf, np.nan
    want[3], want[149] = 0, 0x7fffffff
    assert np.array_equal(Q.qadc_ivf_assign(to_gpu(coarse), to_gpu(x)).cpu().numpy(), want)
    coarse[want[10], 2] = np.inf       # the cell vector 10 was in
    keep = np.isfinite(coarse).all(1)
    fine = np.delete(np.arange(150), [3, 149])
    want[fine] = np.flatnonzero(keep)[_closest(x[fine], coarse[keep])]
    want[3] = 0 if np.isfinite(coarse[0, 5]) else want[3]
    assert np.array_equal(Q.qadc_ivf_assign(to_gpu(coarse), to_gpu(x)).cpu().numpy(), want)


@pytest.mark.parametrize("d,K,n", [(16, 300, 4_097), (64, 260, 131_073), (100, 90, 700), (128, 257, 131_500), (250, 130, 600),
                                   (32, 200, 98_304), (32, 1_030, 49_200), (48, 70, 98_310), (64, 256, 49_152), (96, 90, 98_305),
                                   (96, 300, 49_151), (100, 1_024, 98_400), (24, 4_100, 98_320), (8, 4_097, 98_304), (256, 260, 49_155)])
@pytest.mark.parametrize("kind", ["range", "clusters", "crowds", "same samples", "runs of NaN"])
def test_ivf_assign_where_the_filter_must_give_up(Q, d, K, n, kind):
    """What 11-bit factors cannot tell or hold is left to the routes behind them: vectors and centroids beyond their range
    and below it, clusters far apart of cells close together, three to eight cells as close as each other, a scale guessed
    from centroids that are all the same, 40 centroids of NaN in a row."""
    rng = np.random.default_rng(d + K)
    coarse, x = rng.normal(size=(K, d)), rng.normal(size=(n, d))
    if kind == "range":
        coarse[::7] *= 10.0 ** rng.uniform(-8, 8, size=(len(coarse[::7]), 1))
        x[::5] *= 10.0 ** rng.uniform(-8, 8, size=(len(x[::5]), 1))
    elif kind == "clusters":
        far = 300.0 * rng.normal(size=(4, d))
        coarse, x = coarse + far[rng.integers(0, 4, K)], x + far[rng.integers(0, 4, n)]
    elif kind == "crowds":
        copies = 3 + np.arange(K) % 6
        coarse = np.repeat(coarse, copies, axis=0)[rng.permutation(K)]
        coarse += 1e-6 * rng.integers(0, 2, size=coarse.shape)
    elif kind == "same samples":
        coarse[[k * K // 8 for k in range(8)]] = coarse[0]
        coarse *= 1e-3
    coarse, x = coarse.astype(np.float32), x.astype(np.float32)
    keep = np.arange(K)
    if kind == "runs of NaN":
        coarse[20:60, d // 2] = np.nan
        keep = np.flatnonzero(np.isfinite(coarse).all(1))
    got = Q.qadc_ivf_assign(to_gpu(coarse), to_gpu(x)).cpu().numpy()
    some = np.arange(n) if n < 5000 else np.concatenate([np.arange(0, n, 29), np.arange(n - 500, n)])   # (the host takes minutes for all)
    assert np.array_equal(got[some], keep[_closest(x[some], coarse[keep])])


def test_ivf_assign_unaligned_rows(Q):
    """Rows and centroids that start 4 bytes off a 16-byte boundary."""
    rng = np.random.default_rng(9)
    coarse, x = rng.uniform(0, 1, size=(50, 64)).astype(np.float32), rng.uniform(0, 1, size=(333, 64)).astype(np.float32)
    gc = to_gpu(np.concatenate([[0.0], coarse.ravel()]).astype(np.float32))[1:].view(50, 64)
    gx = to_gpu(np.concatenate([[0.0], x.ravel()]).astype(np.float32))[1:].view(333, 64)
    assert np.array_equal(Q.qadc_ivf_assign(gc, gx).cpu().numpy(), _closest(x, coarse))


@pytest.mark.parametrize("K,n", [(1000, 100_003), (1, 5000), (65536, 300_000), (48, 63), (7, 0), (300, 4096 * 3 + 1)])
def test_ivf_group_is_the_stable_grouping(Q, O, K, n):
    import torch
    from workloads import zipf_list_sizes
    rng = np.random.default_rng(K + n)
    if n:
        sizes = zipf_list_sizes(n, K, 0.8, 1) if K > 1 else np.array([n])
        cells = np.repeat(np.arange(K), sizes).astype(np.int32)[:n]
        if len(cells) < n:
            cells = np.concatenate([cells, rng.integers(0, K, size=n - len(cells)).astype(np.int32)])
        rng.shuffle(cells)
    else:
        cells = np.zeros(0, dtype=np.int32)
    nbytes = Q.qadc_ivf_group_workspace_bytes(n, K)
    ws = torch.full((max(nbytes, 16),), 0xAB, dtype=torch.uint8, device="cuda:0")   # dirty on purpose
    g = to_gpu(cells) if n else torch.zeros((0,), dtype=torch.int32, device="cuda:0")
    for _ in range(2):   # the workspace is reused as the first call left it
        list_off, ids = Q.qadc_ivf_group(g, K, workspace=ws)
        want_off = np.zeros(K + 1, dtype=np.int64)
        np.cumsum(np.bincount(cells, minlength=K), out=want_off[1:])
        assert np.array_equal(list_off.cpu().numpy(), want_off)
        assert np.array_equal(idx_np(ids), np.argsort(cells, kind="stable").astype(np.uint32))


def test_ivf_group_leaves_out_cells_out_of_range(Q):
    rng = np.random.default_rng(4)
    K, n = 50, 10_000
    cells = rng.integers(0, K, size=n).astype(np.int32)
    cells[::7] = -1
    cells[3::11] = K + 5
    ok = (cells >= 0) & (cells < K)
    list_off, ids = Q.qadc_ivf_group(to_gpu(cells), K)
    want_off = np.zeros(K + 1, dtype=np.int64)
    np.cumsum(np.bincount(cells[ok], minlength=K), out=want_off[1:])
    assert np.array_equal(list_off.cpu().numpy(), want_off)
    kept = np.flatnonzero(ok)
    want = kept[np.argsort(cells[kept], kind="stable")].astype(np.uint32)
    assert np.array_equal(idx_np(ids)[:len(want)], want)


@pytest.mark.parametrize("m", [16, 32])
def test_index_built_on_the_gpu_equals_the_oracles(Q, O, m):
    """assign -> group -> encode on the GPU give the oracle's index byte for byte, and a search of it
    gives the oracle's search of the oracle's index."""
    import torch
    coarse, cb, x, index = build_ivf(O, n=30_000, K=40, m=m, seed=10 + m)
    gx, gco, gcb = to_gpu(x), to_gpu(coarse), to_gpu(cb)
    cells = Q.qadc_ivf_assign(gco, gx)
    list_off, ids = Q.qadc_ivf_group(cells, len(coarse))
    codes = Q.qadc_ivf_encode(gco, gcb, gx, cells, ids)
    assert np.array_equal(list_off.cpu().numpy(), index["list_off"])
    assert np.array_equal(idx_np(ids), index["ids"])
    assert np.array_equal(codes.cpu().numpy(), index["codes"])
    gix = Q.IvfIndex(gco, list_off, codes, ids, gcb)
    rng = np.random.default_rng(1)
    queries = (x[rng.integers(0, len(x), size=6)] + rng.normal(scale=6, size=(6, x.shape[1]))).astype(np.float32)
    got_ids, dist, probes, qluts = Q.qadc_ivf_search(gix, to_gpu(queries), 6, 50, 300, debug=True)
    torch.cuda.synchronize()
    for iq in range(len(queries)):
        rep = O.ivf_quick_adc_search(index, coarse, cb, queries[iq], 6, 300, 50,
                                     probes=probes[iq].cpu().numpy(), qluts=qluts[iq].cpu().numpy())
        assert np.array_equal(idx_np(got_ids)[iq], rep["ids"])
        assert np.array_equal(dist[iq].cpu().numpy(), rep["dist"])


def test_ivf_encode_guards_ids_and_cells(Q, O):
    import torch
    coarse, cb, x, index = build_ivf(O, n=6000, K=8, seed=3)
    cells = O.ivf_assign(x, coarse).astype(np.int32)
    ids = np.arange(len(x), dtype=np.uint32)
    cells_bad = cells.copy()
    cells_bad[5] = 99
    ids_bad = ids.copy()
    ids_bad[9] = 4_000_000_000
    codes = Q.qadc_ivf_encode(to_gpu(coarse), to_gpu(cb), to_gpu(x), to_gpu(cells_bad),
                              to_gpu(ids_bad.view(np.int32))).cpu().numpy()
    from oracle import cref
    want = cref.pq_encode((x - coarse[cells]).astype(np.float32), cb)
    want[5] = 0
    want[9] = 0
    assert np.array_equal(codes, want)


# ------------------------------------------------------------------ k-means

@pytest.mark.parametrize("n,d,m,ksub", [(1, 4, 4, 16), (700, 6, 2, 16), (8191, 8, 4, 16), (8192, 8, 4, 16), (8193, 130, 1, 16),
                                        (20_001, 24, 8, 64), (17_000, 96, 8, 256), (9_000, 130, 2, 16)])
def test_pq_train_means_are_row_order_float64_sums(Q, O, n, d, m, ksub):
    """One update from known labels, bit for bit: sums in row order in float64, one division, one rounding; a
    centroid that owns nothing keeps its value.  Sizes around a round of labels (8192), a stage of rows and a
    workgroup's 64 components; one centroid owns most of the rows."""
    rng = np.random.default_rng(n + d)
    x = rng.uniform(0, 255, size=(n, d)).astype(np.float32)
    x[n // 3:] = (x[n // 3:n // 3 + 1] + rng.normal(scale=3, size=(n - n // 3, d))).astype(np.float32)
    rows = np.minimum(rng.permutation(max(n, ksub))[:ksub], n - 1).astype(np.int64)   # n < ksub: repeated rows, centroids that own nothing
    dsub = d // m
    start = np.stack([x[rows, j * dsub:(j + 1) * dsub] for j in range(m)])
    want = start.copy()
    labels = O.pq_encode(x, start)
    for j in range(m):
        for i in range(ksub):
            own = np.flatnonzero(labels[:, j] == i)
            if len(own):
                sums = np.cumsum(x[own, j * dsub:(j + 1) * dsub].astype(np.float64), axis=0)[-1]   # cumsum: strictly in order
                want[j, i] = (sums / len(own)).astype(np.float32)
    got = Q.qadc_pq_train(to_gpu(x), m, ksub, to_gpu(rows), 1).cpu().numpy()
    assert np.array_equal(got, want)


@pytest.mark.parametrize("n,d", [(2, 1), (4_096, 4), (4_097, 4), (8_192, 64), (8_193, 2), (20_479, 3), (20_480, 64), (20_481, 65), (40_961, 5)])
def test_pq_train_means_where_the_order_of_the_sum_decides(Q, n, d):
    """All rows with the first centroid (repeated starting rows, ties to the lowest index) and components whose float64
    sum depends on the order of the additions, a mean half way between two float32, infinities and NaN: still the
    row-order sum, bit for bit.  Sizes around the forms of the kernel
    (4096, 8192), a round of labels (20,480) and a workgroup's 64 components."""
    rng = np.random.default_rng(n)
    x = (rng.normal(size=(n, d)) * 10.0 ** rng.uniform(-12, 12, size=(n, d))).astype(np.float32)
    x[:, 0] = 1.0
    x[::2, 0] = np.float32(1.0) + np.float32(2.0 ** -23)    # n even: the mean is 1 + 2^-24
    if d > 4:
        x[5, 1], x[6, 2], x[7, 2], x[9, 3] = np.inf, np.inf, -np.inf, np.nan
        x[:, 4] = -0.0
    rows = np.zeros(16, dtype=np.int64)
    got = Q.qadc_pq_train(to_gpu(x), 1, 16, to_gpu(rows), 1).cpu().numpy()
    with np.errstate(all="ignore"):
        want = (np.cumsum(np.vstack([np.zeros((1, d)), x.astype(np.float64)]), axis=0)[-1] / n).astype(np.float32)
    assert np.array_equal(got[0, 0], want, equal_nan=True)
    assert np.array_equal(np.signbit(got[0, 0]), np.signbit(want)) or np.isnan(want).any()
    assert np.array_equal(got[0, 1:], np.broadcast_to(x[0], (15, d)))


@pytest.mark.parametrize("per_round", [1, 2, 5])
@pytest.mark.parametrize("tiny", [2.0 ** -54, 3 * 2.0 ** -54, -(2.0 ** -55)])
def test_pq_train_means_of_rows_far_apart(Q, per_round, tiny):
    """256 rows of a centroid, a few per round of 20,480 labels, so that the first chains of the parallel sum are as long as there
    are rounds; in row order all but two of them vanish in the sum and the mean is half way between two float32."""
    c, rounds = 256, -(-256 // per_round)
    x = np.full((rounds * 20_480, 1), 1000.0, dtype=np.float32)
    at = np.concatenate([r * 20_480 + 7 + 11 * np.arange(per_round) for r in range(rounds)])[:c]
    x[at, 0] = tiny
    x[at[0], 0], x[at[1], 0] = 1.0, 2.0 ** -24
    rows = np.full(16, 0, dtype=np.int64)
    rows[0] = at[0]
    got = Q.qadc_pq_train(to_gpu(x), 1, 16, to_gpu(rows), 1).cpu().numpy()
    want = np.float32(np.cumsum(x[at, 0].astype(np.float64))[-1] / c)
    assert got[0, 0, 0] == want and np.all(got[0, 1:] == 1000.0)


def _codes_by_definition(x, cb):
    """enc(x) from float64 distances summed in increasing component order, ties to the lowest index; u8 [n][m]."""
    m, k, dsub = cb.shape
    out = np.empty((len(x), m), dtype=np.uint8)
    with np.errstate(all="ignore"):
        for j in range(m):
            acc = np.zeros((len(x), k))
            for t in range(dsub):
                df = x[:, j * dsub + t, None].astype(np.float64) - cb[j, None, :, t].astype(np.float64)
                acc = acc + df * df
            acc[np.isnan(acc)] = np.inf
            out[:, j] = np.argmin(acc, axis=1)
    return out


def _pack(comps, k):
    n, m = comps.shape
    if k == 256:
        return comps
    bits = 4 if k == 16 else 6
    v = np.zeros((n, bits * m), dtype=np.uint8)
    for b in range(bits):
        v[:, b::bits] = (comps >> b) & 1
    return np.packbits(v.reshape(n, -1, 8), axis=2, bitorder="little")[:, :, 0]


@pytest.mark.parametrize("n,m,dsub,k", [(1, 2, 8, 16), (63, 6, 1, 16), (65, 10, 4, 16), (257, 16, 5, 16), (700, 18, 16, 16),
                                        (130, 8, 30, 16), (190, 8, 3, 64), (61, 12, 12, 64), (129, 4, 17, 64),
                                        (100, 1, 2, 256), (66, 7, 12, 256), (321, 8, 6, 256), (64, 5, 40, 256)])
def test_pq_encode_where_float32_cannot_tell(Q, n, m, dsub, k):
    """Near ties around the float32 margin, exact ties, and values at both ends of the float32 range, infinities and
    NaN included: the codes are those of the float64 definition; rows and bytes around a wavefront's share; an output
    that starts at an odd address."""
    import torch
    rng = np.random.default_rng(n * m + k)
    cb = rng.uniform(0, 255, size=(m, k, dsub)).astype(np.float32)
    cb[:, k // 2] = cb[:, k // 3]                                                   # the lower index wins
    cb[:, k // 4] = np.nextafter(cb[:, k // 5], np.float32(1e9))                   # one unit in the last place apart
    x = rng.uniform(0, 255, size=(n, m * dsub)).astype(np.float32)
    own = rng.integers(0, k, size=(n, m))
    near = np.concatenate([cb[j][own[:, j]] for j in range(m)], axis=1)
    mid = np.concatenate([(cb[j][own[:, j]] + cb[j][(own[:, j] + 1) % k]) / 2 for j in range(m)], axis=1).astype(np.float32)
    kind = rng.integers(0, 8, size=n)
    x[kind == 1] = near[kind == 1]
    x[kind == 2] = mid[kind == 2]                                                   # as far from two centroids
    x[kind == 3] = near[kind == 3] + np.float32(1e-3)
    x[kind == 4] *= np.float32(1e17)                                                # squares leave the float32 range
    x[kind == 5, 0] = np.inf
    x[kind == 6, -1] = np.nan
    if n > 300:
        cb[m - 1] *= np.float32(1e-22)                                              # squares below the normal range
        x[kind == 7, -dsub:] *= np.float32(1e-22)
        cb[0, k - 1, 0] = np.inf
        cb[0, 0, -1] = np.nan
    want = _pack(_codes_by_definition(x, cb), k)
    flat = torch.zeros((n * want.shape[1] + 1,), dtype=torch.uint8, device="cuda:0")
    for out in (flat[1:].view(n, -1), flat[:-1].view(n, -1)):
        got = Q.qadc_pq_encode(to_gpu(cb), to_gpu(x), out=out)
        assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("n,K", [(100_003, 256), (300_000, 4096), (1_000_000, 5_998)])
def test_group_with_the_smallest_workspace(Q, n, K):
    """Fewer, longer parts where the workspace holds no more counters: the same grouping.  A workspace for K cells also
    serves fewer cells."""
    import torch
    from gpu_common import smallest_workspace
    cells = to_gpu(np.random.default_rng(n).integers(0, K, size=n).astype(np.int32))
    want = Q.qadc_ivf_group(cells, K)
    least, got = smallest_workspace(Q, lambda ws: Q.qadc_ivf_group(cells, K, workspace=ws))
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert least <= Q.qadc_ivf_group_workspace_bytes(n, K)
    fewer = cells % (K - 28)
    ws = torch.empty((Q.qadc_ivf_group_workspace_bytes(n, K),), dtype=torch.uint8, device="cuda:0")
    got, want = Q.qadc_ivf_group(fewer, K - 28, workspace=ws), Q.qadc_ivf_group(fewer, K - 28)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    if K < 5000:
        want = Q.qadc_multi_index_group(cells, K)
        _, got = smallest_workspace(Q, lambda ws: Q.qadc_multi_index_group(cells, K, workspace=ws))
        assert all(torch.equal(a, b) for a, b in zip(got, want))


# every compiled length of a sub-vector, and the general form's blocks of 8, 4, 2 and 1 components with and without rests
@pytest.mark.parametrize("dsub", list(range(1, 22)) + [22, 23, 24, 27, 28, 31, 32, 33])
@pytest.mark.parametrize("k", [16, 64, 256])
def test_pq_encode_lengths_of_sub_vectors(Q, dsub, k):
    test_pq_encode_where_float32_cannot_tell(Q, 330, 4, dsub, k)


@pytest.mark.parametrize("dsub,m", [(8, 8), (11, 6), (21, 4), (23, 2)])
def test_residual_codes_of_ties(Q, dsub, m):
    """Residuals that are zero, or as far from two centroids, in whole wavefronts: the float64 walk on differences."""
    rng = np.random.default_rng(dsub)
    d, n, K = dsub * m, 1000, 7
    coarse = rng.integers(0, 9, size=(K, d)).astype(np.float32)
    cb = rng.integers(-2, 3, size=(m, 16, dsub)).astype(np.float32)
    cb[0, 3] = cb[0, 9]
    cells = rng.integers(0, K, size=n).astype(np.int32)
    x = coarse[cells] + rng.integers(-2, 3, size=(n, d)).astype(np.float32)
    x[:200] = coarse[cells[:200]]
    ids = rng.permutation(n).astype(np.int32)
    got = Q.qadc_ivf_encode(to_gpu(coarse), to_gpu(cb), to_gpu(x), to_gpu(cells), to_gpu(ids))
    want = _pack(_codes_by_definition((x - coarse[cells])[ids], cb), 16)
    assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("k,m,dsub", [(16, 16, 5), (16, 16, 8), (16, 8, 24), (64, 8, 8), (256, 8, 8), (256, 8, 10)])
def test_pq_encode_of_ties_is_not_much_slower(Q, k, m, dsub):
    """Components that are zero everywhere (padded vectors), repeated centroids: every sub-vector needs float64.  That costs
    a second walk over the centroids, not fifty."""
    import torch
    from gpu_common import gpu_us
    g = torch.Generator(device="cuda:0")
    g.manual_seed(k)
    x = torch.randn((200_000, m * dsub), generator=g, device="cuda:0")
    cb = torch.randn((m, k, dsub), generator=g, device="cuda:0")
    usual = gpu_us(lambda: Q.qadc_pq_encode(cb, x), reps=5)
    twice = cb.clone()
    twice[:, k // 2:] = cb[:, :k // 2]
    assert gpu_us(lambda: Q.qadc_pq_encode(twice, x), reps=5) < 8 * usual
    x[:] = 0
    cb[:] = 0
    assert gpu_us(lambda: Q.qadc_pq_encode(cb, x), reps=5) < 8 * usual


# (131,072 vectors and more in aligned rows of 32, 64, 96 or 128 components take the kernel of 512 threads)
@pytest.mark.parametrize("d,K,n", [(32, 300, 131_500), (64, 70, 131_200), (96, 500, 131_072), (128, 333, 131_111),
                                   (4, 900, 5_000), (16, 200, 3_000), (20, 128, 9_999), (100, 64, 1_300), (200, 97, 2_000),
                                   (256, 60, 700), (128, 40, 1)])
@pytest.mark.parametrize("kind", ["lattice", "near", "repeats", "stray", "nan"])
def test_ivf_assign_of_crowded_cells(Q, d, K, n, kind):
    """More close cells than a lane of the filter remembers, in one half of its lanes or both; a few centroids far away
    or not finite, which may not loosen or spoil the choice among the others."""
    import torch
    rng = np.random.default_rng(d + K + n)
    coarse = rng.integers(0, 3, size=(K, d)).astype(np.float32)
    x = rng.integers(0, 3, size=(n, d)).astype(np.float32)
    if kind == "near":
        coarse += rng.normal(size=(K, d)).astype(np.float32) * np.float32(1e-4)
    if kind == "repeats":
        coarse = coarse[rng.integers(0, max(1, K // 5), size=K)]
        x[::3] = coarse[rng.integers(0, K, size=len(x[::3]))]
    if kind in ("stray", "nan"):
        coarse[::9] *= np.float32(1e6)
        coarse[K // 2] = np.float32(3e19)
        coarse[K // 3] = np.inf
    if kind == "nan":
        coarse[1::3, 0] = np.nan
        coarse[1::3, -1] = np.nan
        x[n // 2] = np.float32(1e20)
    g, got = to_gpu(coarse).double(), Q.qadc_ivf_assign(to_gpu(coarse), to_gpu(x))
    want = torch.empty_like(got)
    for s in range(0, n, 2048):
        xx = to_gpu(x[s:s + 2048]).double()
        dist = torch.zeros((len(xx), K), dtype=torch.float64, device="cuda:0")
        for t in range(d):  # in increasing component order; a fused step rounds once, as close calls may need
            dist = torch.addcmul(dist, xx[:, t, None] - g[None, :, t], xx[:, t, None] - g[None, :, t])
        dist = torch.where(dist.isnan(), torch.inf, dist)
        want[s:s + 2048] = (dist == dist.min(1, keepdim=True).values).int().argmax(1).int()
    assert torch.equal(got, want)


# split factors (few vectors) are merged every 512 cells, binary16 factors every 4096; the workgroups of 512 threads from 32,768
# (d = 256), 65,536 and 98,304 vectors (d = 32)
@pytest.mark.parametrize("d,K,n", [(128, 511, 700), (64, 513, 700), (200, 1540, 500), (32, 1030, 900),
                                   (64, 4095, 50_001), (128, 4097, 50_001), (128, 4099, 65_601), (64, 8193, 65_536),
                                   (256, 4100, 32_801), (32, 4096, 98_400), (96, 12_300, 66_000), (24, 4_200, 99_000)])
def test_ivf_assign_over_many_cells(Q, d, K, n):
    """The closest cell, and the lowest of equal ones, in any of the stretches of cells whose finds are merged: whole numbers,
    whose squares and sums float64 holds exactly."""
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(d + K + n)
    coarse = torch.randint(0, 60, (K, d), generator=g, device="cuda:0").float()
    coarse[K - K // 5:] = coarse[:K // 5]                                # the same centroids, far apart
    coarse[K // 2] = coarse[K - 1]
    x = coarse[torch.randint(0, K, (n,), generator=g, device="cuda:0")]
    x = x + torch.randint(-20, 21, (n, d), generator=g, device="cuda:0").float()
    got = Q.qadc_ivf_assign(coarse, x)
    c = coarse.double()
    for s in range(0, n, 8192):
        dist = (c * c).sum(1)[None] - 2 * (x[s:s + 8192].double() @ c.T)
        want = (dist == dist.min(1, keepdim=True).values).int().argmax(1).int()
        assert torch.equal(got[s:s + 8192], want)


# split factors in phases: aligned rows from 32,769 vectors on or beyond 128 components, others from 65 components on; the block on the
# other side of the line
@pytest.mark.parametrize("d,K,n", [(128, 513, 32_769), (128, 1031, 32_768), (64, 1540, 33_000), (32, 520, 32_800), (96, 33, 40_001),
                                   (256, 1057, 700), (65, 515, 900), (100, 1025, 33_001), (255, 40, 130), (63, 1030, 33_000)])
def test_ivf_assign_of_split_factors_in_phases(Q, d, K, n):
    test_ivf_assign_over_many_cells(Q, d, K, n)


# 512 vectors per workgroup from 4096 cells on, where a row is not whole steps of 16 components or not aligned
@pytest.mark.parametrize("d,K,n", [(33, 4096, 98_304), (47, 4109, 98_401), (64, 4095, 98_305), (65, 4097, 99_001), (95, 8193, 98_815)])
def test_ivf_assign_of_unaligned_rows_by_wide_workgroups(Q, d, K, n):
    test_ivf_assign_over_many_cells(Q, d, K, n)


@pytest.mark.parametrize("K,dh,n", [(2, 4, 1_000), (64, 16, 4_000), (333, 32, 131_500)])
def test_multi_index_assign_of_crowded_cells(Q, K, dh, n):
    """Both halves leave vectors to the second kernel, which finds them among the cells of the first half."""
    import torch
    rng = np.random.default_rng(K)
    halves = rng.integers(0, 2, size=(2, K, dh)).astype(np.float32)
    halves[:, K // 2:] = halves[:, :K - K // 2]
    x = rng.integers(0, 2, size=(n, 2 * dh)).astype(np.float32)
    got = Q.qadc_multi_index_assign(to_gpu(halves), to_gpu(x)).cpu().numpy()
    want = np.zeros(n, np.int64)
    for h in range(2):
        xx = x[:, h * dh:(h + 1) * dh]
        dist = (xx ** 2).sum(1)[:, None] - 2 * xx @ halves[h].T + (halves[h] ** 2).sum(1)[None]  # whole numbers: exact
        want = want * K + dist.argmin(1)
    assert np.array_equal(got, want)


# the last tile of the filter has one to 24 places past the last cell, or 31; aligned rows and others; split factors from the start,
# and behind binary16 ones (50,000 vectors, most of them with more rivals than a lane remembers)
@pytest.mark.parametrize("d,K,n", [(128, 127, 600), (128, 300, 600), (32, 488, 600), (64, 255, 600), (256, 506, 300),
                                   (100, 127, 600), (200, 500, 300), (17, 225, 600), (3, 95, 600), (128, 300, 50_000),
                                   (64, 511, 50_000)])
@pytest.mark.parametrize("last", [1e34, 1e36, 1e37, -1e38, 3e38])
def test_ivf_assign_with_a_last_centroid_far_out(Q, d, K, n, last):
    """Nothing of the last centroid's shows in the places past it, whose scores are no candidates: the ordinary cells win."""
    rng = np.random.default_rng(K + n)
    coarse = rng.integers(-9, 10, size=(K, d)).astype(np.float32)
    if n >= 50_000:
        coarse[:K // 2] = coarse[K // 2:2 * (K // 2)]
        coarse[:K // 4] = coarse[K // 4:2 * (K // 4)]
        coarse[:K // 8] = coarse[K // 8:2 * (K // 8)]
    coarse[K - 1] = 0
    coarse[K - 1, d // 3] = last
    x = (coarse[rng.integers(0, K - 1, size=n)] + rng.integers(-2, 3, size=(n, d))).astype(np.float32)
    near = coarse[:K - 1].astype(np.float64)
    want = np.concatenate([((near * near).sum(1)[None] - 2 * xx.astype(np.float64) @ near.T).argmin(1)  # whole numbers: exact
                           for xx in np.array_split(x, max(1, n // 5000))])
    assert np.array_equal(Q.qadc_ivf_assign(to_gpu(coarse), to_gpu(x)).cpu().numpy(), want)
    halves = np.stack([coarse, coarse[::-1]])       # (the far centroid first in the second half)
    got = Q.qadc_multi_index_assign(to_gpu(halves), to_gpu(np.concatenate([x, x[::-1]], axis=1))).cpu().numpy()
    # the second half's cells in reverse order: the lowest of equal ones is the last there
    other = np.concatenate([((near * near).sum(1)[None] - 2 * xx.astype(np.float64) @ near.T)[:, ::-1].argmin(1)
                            for xx in np.array_split(x[::-1], max(1, n // 5000))]) + 1
    assert np.array_equal(got, want * K + other)


def _with_copies(kind, c, rng):
    """Centroids of which most are copies of others."""
    K = len(c)
    i = np.arange(K)
    if kind == "one":
        return c[i * 0]
    if kind == "last_differs":
        return c[np.where(i == K - 1, 1, 0)]
    if kind == "first_differs":
        return c[np.where(i == 0, 1, 0)]
    if kind == "alternating":
        return c[i % 2]
    if kind == "padded_in_front":
        return c[np.where(i < K // 2, K // 2, i)]
    if kind == "eight_times":
        return c[i % max(1, K // 8)]
    return c[rng.integers(0, min(K, 20), size=K)]  # any_order


# (copies are looked for where more than 20 of a workgroup's vectors, or more than 128 of up to four components, are left to the definition; a
# sample of 256 rows from 257 cells on, at most 65,536 cells, of which 4096 are listed)
@pytest.mark.parametrize("d,K,n", [(16, 3, 300), (64, 256, 700), (128, 257, 5_000), (100, 700, 3_000), (2, 900, 2_000), (200, 300, 900),
                                   (256, 290, 600), (64, 1024, 70_000), (8, 40_000, 300), (4, 65_537, 400), (17, 5_000, 600)])
@pytest.mark.parametrize("kind", ["one", "last_differs", "first_differs", "alternating", "padded_in_front", "eight_times", "any_order"])
def test_ivf_assign_with_copies_of_centroids(Q, d, K, n, kind):
    """The lowest of equal cells, wherever the copies stand; two columns with both zeros, and rows of NaN that are copies."""
    rng = np.random.default_rng(d + K)
    first = rng.integers(-3, 4, size=(K, d)).astype(np.float32)
    coarse = _with_copies(kind, first, rng)
    if kind in ("alternating", "any_order"):
        coarse[K // 3, 0] = coarse[K // 2, -1] = np.float32(-0.0)
    if kind == "eight_times" and K > 100:
        coarse[K // 8:K // 7] = np.nan
    x = (coarse[rng.integers(0, K, size=n)] + rng.integers(-1, 2, size=(n, d))).astype(np.float32)
    x = np.where(np.isnan(x), 0, x).astype(np.float32)
    c = np.where(np.isnan(coarse), np.inf, coarse)
    wanted = []
    for xx in np.array_split(x.astype(np.float64), max(1, n * K // 20_000_000)):
        cc = np.where(np.isinf(c), 0, c).astype(np.float64)
        dist = (xx * xx).sum(1)[:, None] - 2 * xx @ cc.T + (cc * cc).sum(1)[None]  # whole numbers: exact
        wanted.append(np.where(np.isinf(c).any(1)[None], np.inf, dist).argmin(1))
    assert np.array_equal(Q.qadc_ivf_assign(to_gpu(coarse), to_gpu(x)).cpu().numpy(), np.concatenate(wanted))


@pytest.mark.parametrize("d,K", [(128, 256), (64, 1024), (200, 300), (128, 4096)])
@pytest.mark.parametrize("kind", ["one", "last_differs", "first_differs", "alternating", "padded_in_front", "eight_times", "any_order"])
def test_ivf_assign_is_not_slowed_by_copies_of_centroids(Q, d, K, kind):
    """Copies cost a search for them and the filter's passes in vain, not an exact pass over all cells (up to 37 times the usual)."""
    import torch
    from gpu_common import gpu_us
    rng = np.random.default_rng(d)
    coarse = (30 * rng.normal(size=(K, d))).astype(np.float32)
    x = to_gpu((coarse[rng.integers(0, K, size=200_000)] + 18 * rng.normal(size=(200_000, d))).astype(np.float32))
    usual = gpu_us(lambda c=to_gpu(coarse): Q.qadc_ivf_assign(c, x), reps=5)
    us = gpu_us(lambda c=to_gpu(_with_copies(kind, coarse, rng)): Q.qadc_ivf_assign(c, x), reps=5)
    assert us < 12 * usual, (us, usual)


@pytest.mark.parametrize("d,K", [(128, 256), (64, 1024), (200, 300)])
def test_ivf_assign_is_not_slowed_by_a_few_centroids(Q, d, K):
    """One stray centroid, one that is not finite, all of them twice: not much slower than without."""
    import torch
    from gpu_common import gpu_us
    g = torch.Generator(device="cuda:0")
    g.manual_seed(d)
    coarse = 30 * torch.randn((K, d), generator=g, device="cuda:0")
    x = coarse[torch.randint(0, K, (200_000,), generator=g, device="cuda:0")] + 18 * torch.randn((200_000, d), generator=g,
                                                                                                device="cuda:0")
    usual = gpu_us(lambda: Q.qadc_ivf_assign(coarse, x), reps=5)
    for change, limit in ((lambda c: c[K // 3].mul_(100), 2), (lambda c: c[K // 5].fill_(float("nan")), 2),
                          (lambda c: c[K // 2:].copy_(c[:K // 2]), 4.5), (lambda c: c.copy_(c[:1].expand(K, d).clone()), 14)):
        c = coarse.clone()
        change(c)
        us = gpu_us(lambda: Q.qadc_ivf_assign(c, x), reps=5)
        assert us < limit * usual, (us, usual)


@pytest.mark.parametrize("n", [1, 3, 129, 131, 255, 2049, 4097, 8191, 8194, 20479, 20482, 21001, 40963])
@pytest.mark.parametrize("dsub", [1, 3, 8, 64])
def test_pq_train_finds_every_row_of_a_centroid(Q, n, dsub):
    """Whole numbers (every sum is exact in float64): the means are those of the rows, at the ends of a word of labels, of a
    wavefront's share and of a round; columns of labels that do not start on a word; one centroid that owns nearly all rows."""
    rng = np.random.default_rng(n * 100 + dsub)
    m = 3
    own = np.where(rng.random((n, m)) < 0.8, 5, rng.integers(0, 16, (n, m)))
    own[0] = 5
    own[-1] = 15
    # component 0 says which centroid; the others are noise of whole numbers, smaller than the distance of two centroids
    x = rng.integers(-3, 4, (n, m, dsub)).astype(np.float32)
    x[:, :, 0] += 1024.0 * own
    for c in range(min(n, 16)):  # rows that name every centroid, where there are as many
        own[c] = (5 + c) % 16 if n >= 16 else own[c]
    if n >= 16:
        x[:16, :, 0] = 1024.0 * own[:16]
    rows = np.array([min(c, n - 1) for c in range(16)], dtype=np.int64)
    cb0 = x[rows]                                            # [16][m][dsub]
    want = np.empty((m, 16, dsub), dtype=np.float32)
    for j in range(m):
        dist = ((x[:, j, None, :].astype(np.float64) - cb0[None, :, j, :]) ** 2).sum(-1) if n <= 4097 else None
        if dist is None:
            order = np.argsort(cb0[:, j, 0], kind="stable")  # one centroid per value of component 0 (n >= 16)
            label = order[np.rint(x[:, j, 0] / 1024).astype(int)]
        else:
            label = dist.argmin(1)
        for i in range(16):
            r = x[label == i, j].astype(np.float64)
            want[j, i] = (r.sum(0) / len(r)).astype(np.float32) if len(r) else cb0[i, j]
    got = Q.qadc_pq_train(to_gpu(x.reshape(n, m * dsub)), m, 16, to_gpu(rows), 1).cpu().numpy()
    assert np.array_equal(got.reshape(m, 16, dsub), want)
