"""GPU parity: sketch plan and CountSketch (all three variants) against the
oracle, through the C ABI.

Bar: bit-exact for the plan (integers) and for the deterministic sorted mode;
normwise relative 1e-12 (FP64) / 1e-5 (FP32) for the atomic and LDS modes,
whose association order differs from the sequential fold.
"""
import os

import numpy as np
import pytest

import synth
from gpu_util import bits_equal, rel, to_dev, to_host

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "canonical_fold.txt")


@pytest.fixture(scope="module")
def ms():
    import paper_2508_14209_amd as ms
    return ms


def _inputs(d, n, k, seed, dtype=np.float64):
    A = synth.normal_matrix(d, n, seed=seed, dtype=dtype)
    h = synth.bucket_map(d, k, seed=seed)
    s = synth.signs(d, seed=seed)
    return A, h, s


# ------------------------------------------------------------------- plan
@pytest.mark.parametrize("d,k", [(1, 1), (777, 7), (65536, 2048), (300000, 40), (4194304, 8192)])
def test_bucket_plan_bit_exact(ms, orc, d, k):
    print("plan d=%d k=%d" % (d, k), flush=True)
    h = synth.bucket_map(d, k, seed=d % 97)
    cnt, off, perm, ws = ms.bucket_plan(to_dev(h), k)
    ms.check_status(ws)
    off_ref, perm_ref = orc.bucket_plan(h, k)
    assert np.array_equal(to_host(cnt).astype(np.int64), orc.bucket_hist(h, k))
    assert np.array_equal(to_host(off).astype(np.int64), off_ref)
    assert np.array_equal(to_host(perm).astype(np.int64), perm_ref)


def test_bucket_plan_long_bucket_blocked(ms, orc):
    # up to MS_SORTED_BLOCKED_MAX_K buckets the plan is a blocked stable
    # counting sort: a bucket holding most rows is planned exactly
    d, k = 3 * ms.MS_SORTED_MAX_SEGMENT + 5, 2
    h = np.zeros(d, np.int32)
    h[::7] = 1
    cnt, off, perm, ws = ms.bucket_plan(to_dev(h), k)
    ms.check_status(ws)
    off_ref, perm_ref = orc.bucket_plan(h, k)
    assert np.array_equal(to_host(off).astype(np.int64), off_ref)
    assert np.array_equal(to_host(perm).astype(np.int64), perm_ref)


def test_bucket_plan_segment_limit_reported(ms):
    # beyond MS_SORTED_BLOCKED_MAX_K buckets each bucket is sorted in LDS: one
    # longer than the limit is reported, not mis-sorted
    k = ms.MS_SORTED_BLOCKED_MAX_K + 1
    d = 3 * ms.MS_SORTED_MAX_SEGMENT
    h = (np.arange(d, dtype=np.int64) % k).astype(np.int32)
    h[::2] = 0
    cnt, off, perm, ws = ms.bucket_plan(to_dev(h), k)
    with pytest.raises(ms.MsketchError) as e:
        ms.check_status(ws)
    assert e.value.code == ms.MS_ERR_UNSUPPORTED


# ------------------------------------------------------------------- CountSketch
CASES = [
    # d, n, k, dtype
    (1, 1, 1, np.float64),
    (1000, 3, 64, np.float64),
    (12345, 5, 300, np.float64),   # ragged: k not a power of two, d % 4 != 0
    (65536, 32, 2048, np.float64),  # the 65,536 x 32 FP64, k = 2048 workload
    (12347, 7, 301, np.float32),
    (200000, 9, 4096, np.float32),
    (300, 4, 2000, np.float64),    # k > d: most buckets empty
]


@pytest.mark.parametrize("mode", ["sorted", "lds", "atomic"])
@pytest.mark.parametrize("d,n,k,dtype", CASES)
def test_countsketch_parity(ms, orc, mode, d, n, k, dtype):
    print("countsketch mode=%s d=%d n=%d k=%d %s" % (mode, d, n, k, np.dtype(dtype)), flush=True)
    A, h, s = _inputs(d, n, k, seed=d + n + k, dtype=dtype)
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(s), k, mode=mode)
    ms.check_status(ws)
    Yg = to_host(Y)
    Yr = orc.countsketch(A, h, s, k)
    assert Yg.shape == (k, n) and Yg.dtype == dtype
    if mode == "sorted":
        assert bits_equal(Yg, Yr)
    else:
        assert rel(Yg, Yr) <= (1e-12 if dtype == np.float64 else 1e-5)


@pytest.mark.parametrize("mode", ["sorted", "lds"])
def test_countsketch_full_c2_shape(ms, orc, mode):
    # A 4,194,304 x 65 FP64 ([A | b] of the multisketch least-squares workload), k = 8192
    d, n, k = 4194304, 65, 8192
    print("countsketch full d=%d n=%d k=%d mode=%s" % (d, n, k, mode), flush=True)
    A, h, s = _inputs(d, n, k, seed=14209)
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(s), k, mode=mode)
    ms.check_status(ws)
    Yr = orc.countsketch(A, h, s, k)
    if mode == "sorted":
        assert bits_equal(to_host(Y), Yr)
    else:
        assert rel(to_host(Y), Yr) <= 1e-12


@pytest.mark.parametrize("dtype,k", [(np.float64, 32768), (np.float32, 65536), (np.float32, 131072)])
def test_countsketch_bucket_tiles(ms, orc, dtype, k):
    # more buckets than one workgroup's LDS holds: bucket tiles
    d, n = 1 << 20, 3
    print("countsketch tiles k=%d %s" % (k, np.dtype(dtype)), flush=True)
    A, h, s = _inputs(d, n, k, seed=5, dtype=dtype)
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(s), k, mode="lds")
    ms.check_status(ws)
    assert rel(to_host(Y), orc.countsketch(A, h, s, k)) <= (1e-12 if dtype == np.float64 else 1e-5)


@pytest.mark.parametrize("d,n,k,dtype,tiled", [(300001, 20, 65536, np.float32, True),
                                               (1000, 8, 131072, np.float32, True),
                                               (8192 * 3 + 5, 3, 70001, np.float64, True),
                                               (50000, 2, 41000, np.float32, True),
                                               (8192, 1, 61441, np.float64, True),
                                               (200000, 32, 32768, np.float64, False),
                                               (8192 * 3 + 5, 3, 40000, np.float64, False),
                                               (8192, 1, 16385, np.float64, False)])
def test_countsketch_tiled_plan(ms, orc, d, n, k, dtype, tiled):
    # more buckets than one workgroup's LDS holds (k > 16384).  From four
    # bucket tiles up (k > 40960) the rows of each 8192-row block are grouped
    # by bucket tile first and each tile's workgroups visit only their rows;
    # with two tiles every tile's workgroups stream all rows (untiled).
    # Ragged shapes: a partial last block, one block only, bucket counts that
    # are not powers of two, tiles of unequal length.  With the plan the
    # workspace holds it (4 bytes per row, block padded) besides the codes.
    a_dt = ms.MS_F64 if dtype == np.float64 else ms.MS_F32
    nblk = (d + 8191) // 8192
    extra = (ms.workspace_size("countsketch", d=d, n=n, k=k, a_dtype=a_dt, mode="lds")
             - ms.workspace_size("countsketch", d=d, n=n, k=k, a_dtype=a_dt, mode="atomic"))
    if tiled:
        assert extra >= nblk * 8192 * 4
    print("countsketch tiled d=%d n=%d k=%d %s" % (d, n, k, np.dtype(dtype)), flush=True)
    A, h, s = _inputs(d, n, k, seed=9, dtype=dtype)
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(s), k, mode="lds")
    ms.check_status(ws)
    assert rel(to_host(Y), orc.countsketch(A, h, s, k)) <= (1e-12 if dtype == np.float64 else 1e-5)


@pytest.mark.parametrize("d,n,k,dtype", [(100003, 15, 32768, np.float32),
                                         (100003, 16, 32768, np.float64),
                                         (60000, 37, 32768, np.float32),
                                         (2049, 33, 20000, np.float32),
                                         (260, 49, 40000, np.float64)])
def test_countsketch_column_sets(ms, orc, d, n, k, dtype):
    # Several bucket tiles, a workspace of the status block only: no set, whole
    # sets and left-over columns of the 16 groups (two tiles) or 10 (three), dies
    # without rows.
    import torch
    A, h, s = _inputs(d, n, k, seed=n, dtype=dtype)
    print("column sets d=%d n=%d k=%d %s" % (d, n, k, np.dtype(dtype)), flush=True)
    code, _ = ms.pack_sketch(to_dev(h), to_dev(s), k)
    Y = ms.empty_colmajor(k, n, torch.float64 if dtype == np.float64 else torch.float32, "cuda")
    Y.zero_()
    ws = ms.workspace(256, "cuda")
    ms.countsketch_accumulate(to_dev(A), code, k, Y, mode="lds", ws=ws)
    ms.check_status(ws)
    assert rel(to_host(Y), orc.countsketch(A, h, s, k)) <= (1e-12 if dtype == np.float64 else 1e-5)


# The same sets where they are taken (655,360 rows to a die), one row before, and with left-over
# columns, against FP64 sums by torch.
@pytest.mark.parametrize("d,n,k,dtype", [(8 * 655360, 17, 32768, np.float32),
                                         (8 * 655360 - 8, 17, 32768, np.float32),
                                         (8 * 655360 + 13, 33, 20000, np.float32),
                                         (8 * 655360 + 8, 12, 40000, np.float64)])
def test_countsketch_column_sets_many_rows(ms, d, n, k, dtype):
    import torch
    print("column sets d=%d n=%d k=%d %s" % (d, n, k, np.dtype(dtype)), flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    dt = torch.float64 if dtype == np.float64 else torch.float32
    A = torch.randn((n, d), generator=g, device="cuda", dtype=dt).t()
    h = torch.randint(0, k, (d,), generator=g, device="cuda", dtype=torch.int32)
    s = torch.randint(0, 2, (d,), generator=g, device="cuda", dtype=torch.int8) * 2 - 1
    code, _ = ms.pack_sketch(h, s, k)
    Y = ms.empty_colmajor(k, n, dt, "cuda")
    Y.zero_()
    ws = ms.workspace(256, "cuda")
    ms.countsketch_accumulate(A, code, k, Y, mode="lds", ws=ws)
    ms.check_status(ws)
    ref = torch.zeros((k, n), device="cuda", dtype=torch.float64)
    for j in range(0, n, 8):
        ref[:, j:j + 8] = torch.zeros((k, min(8, n - j)), device="cuda",
                                      dtype=torch.float64).index_add_(
            0, h.long(), A[:, j:j + 8].double() * s.double()[:, None])
    err = (Y.double() - ref).norm().item() / ref.norm().item()
    assert err <= (1e-12 if dtype == np.float64 else 1e-5)


@pytest.mark.parametrize("d,n,k,dtype,one", [
    (7679, 3, 65536, np.float32, None), (7680, 2, 131072, np.float64, None),
    (7681, 5, 131072, np.float32, None), (7680 * 21 + 1, 37, 163841, np.float32, None),
    (7680 * 40, 3, 327681, np.float64, None), (100003, 9, 655360, np.float32, None),
    (61441, 3, 65536, np.float64, 1), (61441, 3, 131072, np.float32, 7),
    (30011, 2, 262144, np.float64, 15), (30011, 2, 600000, np.float32, 31)])
def test_countsketch_tile_lists(ms, orc, d, n, k, dtype, one):
    # The lists of 4, 8, 16 and 32 bucket tiles: row blocks that end just before, at
    # and after a plan block's 7680 rows, fewer blocks than teams of waves, shares
    # that leave a column midway, and (one) all rows in one tile, whose lists are
    # longer than what a team takes at a time.
    print("tile lists d=%d n=%d k=%d %s %s" % (d, n, k, np.dtype(dtype), one), flush=True)
    A, h, s = _inputs(d, n, k, seed=d % 97, dtype=dtype)
    if one is not None:
        nbt = 4
        while nbt * 20480 < k:
            nbt *= 2
        kt = -(-k // nbt)
        h = (one * kt + h % (min(kt, k - one * kt))).astype(h.dtype)
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(s), k, mode="lds")
    ms.check_status(ws)
    assert rel(to_host(Y), orc.countsketch(A, h, s, k)) <= (1e-12 if dtype == np.float64 else 1e-5)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_countsketch_tiled_accumulate_row_blocks(ms, orc, dtype):
    # Y += C A over two row blocks (the streaming form of Sec. 7) through the
    # packed codes, with the tiled plan built from the codes in the workspace
    import torch
    d, n, k, split = 150001, 5, 65536, 70001
    a_dt = ms.MS_F64 if dtype == np.float64 else ms.MS_F32
    A, h, s = _inputs(d, n, k, seed=19, dtype=dtype)
    Y = ms.empty_colmajor(k, n, torch.float64 if dtype == np.float64 else torch.float32, "cuda")
    Y.zero_()
    for r0, r1 in ((0, split), (split, d)):
        print("accumulate rows %d..%d" % (r0, r1), flush=True)
        code, _ = ms.pack_sketch(to_dev(h[r0:r1]), to_dev(s[r0:r1]), k)
        ws = ms.workspace(ms.workspace_size("countsketch", d=r1 - r0, n=n, k=k, a_dtype=a_dt), "cuda")
        ms.countsketch_accumulate(to_dev(A[r0:r1]), code, k, Y, mode="lds", ws=ws)
        ms.check_status(ws)
    assert rel(to_host(Y), orc.countsketch(A, h, s, k)) <= (1e-12 if dtype == np.float64 else 1e-5)


def test_countsketch_tiled_range_errors(ms):
    d, n, k = 20000, 2, 32768
    A, h, s = _inputs(d, n, k, seed=3)
    hb = h.copy()
    hb[12345] = k
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(hb), to_dev(s), k, mode="lds")
    with pytest.raises(ms.MsketchError) as e:
        ms.check_status(ws)
    assert e.value.code == ms.MS_ERR_RANGE
    sb = s.copy()
    sb[9000] = 0
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(sb), k, mode="lds")
    with pytest.raises(ms.MsketchError) as e:
        ms.check_status(ws)
    assert e.value.code == ms.MS_ERR_RANGE


@pytest.mark.parametrize("mode", ["sorted", "lds", "atomic"])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("off", [0, 1])
def test_countsketch_strided_lda(ms, orc, mode, dtype, off):
    # leading dimension not a multiple of the vector width, and (off = 1) a
    # first column that starts one element past an aligned address: the
    # vector loads are element-aligned only
    d, n, k = 5001, 3, 128
    print("strided mode=%s %s off=%d" % (mode, np.dtype(dtype), off), flush=True)
    A, h, s = _inputs(d, n, k, seed=9, dtype=dtype)
    big = np.zeros((d + 3, n), dtype=dtype)
    big[off:off + d] = A
    At = to_dev(big)[off:off + d]
    assert At.stride(1) == d + 3
    Y, ws = ms.countsketch_apply(At, to_dev(h), to_dev(s), k, mode=mode)
    ms.check_status(ws)
    Yr = orc.countsketch(A, h, s, k)
    if mode == "sorted":
        assert bits_equal(to_host(Y), Yr)
    else:
        assert rel(to_host(Y), Yr) <= (1e-12 if dtype == np.float64 else 1e-5)


def _golden_cases():
    for line in open(GOLDEN):
        line = line.strip()
        if line and not line.startswith("#"):
            dt, vals, expect = [t.strip() for t in line.split(";")]
            yield dt, [float(v) for v in vals.split(",")], float(expect)


@pytest.mark.parametrize("case", list(_golden_cases()))
def test_sorted_mode_reproduces_canonical_fold(ms, case):
    dt, vals, expect = case
    dtype = np.float64 if dt == "f64" else np.float32
    d = 3 * len(vals)
    A = np.ones((d, 1), dtype=dtype)
    h = np.ones(d, np.int32)
    s = np.ones(d, np.int8)
    for j, v in enumerate(vals):
        i = 3 * j + 1
        h[i] = 0
        A[i, 0], s[i] = (-v, -1) if j % 2 else (v, 1)
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(s), 2, mode="sorted")
    ms.check_status(ws)
    got = float(to_host(Y)[0, 0])
    assert got == expect and np.signbit(got) == np.signbit(expect)


def test_empty_rows_and_columns(ms):
    import torch
    k = 16
    Y, ws = ms.countsketch_apply(ms.empty_colmajor(0, 3, torch.float64),
                                 torch.empty(0, dtype=torch.int32, device="cuda"),
                                 torch.empty(0, dtype=torch.int8, device="cuda"), k)
    ms.check_status(ws)
    assert np.array_equal(to_host(Y), np.zeros((k, 3)))
    Y, ws = ms.countsketch_apply(ms.empty_colmajor(10, 0, torch.float64),
                                 to_dev(np.zeros(10, np.int32)), to_dev(np.ones(10, np.int8)), k)
    ms.check_status(ws)
    assert Y.shape == (k, 0)


@pytest.mark.parametrize("mode", ["sorted", "lds", "atomic"])
def test_range_errors_reported(ms, mode):
    d, n, k = 100, 2, 8
    A, h, s = _inputs(d, n, k, seed=1)
    hb = h.copy()
    hb[37] = k
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(hb), to_dev(s), k, mode=mode)
    with pytest.raises(ms.MsketchError) as e:
        ms.check_status(ws)
    assert e.value.code == ms.MS_ERR_RANGE
    sb = s.copy()
    sb[5] = 0
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(sb), k, mode=mode)
    with pytest.raises(ms.MsketchError) as e:
        ms.check_status(ws)
    assert e.value.code == ms.MS_ERR_RANGE


# The deterministic fold by slices of buckets (one fold thread per slice): d at
# and around a 4096-row block (below one block the other form runs), bucket
# counts at the edges of the slice widths (1, 2 and 4 buckets) and of the range
# that takes them, columns that give one slice per thread, two, and too many,
# few buckets (long runs in every block, some over the counting sort's limit),
# every row in one bucket, and columns that are not 16-byte aligned.  Bit-exact.
@pytest.mark.parametrize("d,n,k,dt,hmap", [
    (4095, 3, 40, np.float64, "uniform"), (4096, 3, 40, np.float64, "uniform"),
    (4097, 5, 4096, np.float64, "uniform"), (8191, 2, 4097, np.float32, "uniform"),
    (8192, 2, 8192, np.float64, "uniform"), (20483, 9, 8193, np.float64, "uniform"),
    (12289, 66, 16384, np.float64, "uniform"), (9001, 130, 2048, np.float32, "uniform"),
    (9001, 130, 8192, np.float64, "uniform"), (9001, 3, 16385, np.float64, "uniform"),
    (50001, 4, 31, np.float64, "uniform"), (50001, 4, 32, np.float32, "uniform"),
    (30001, 2, 512, np.float64, "one"), (30001, 2, 5000, np.float32, "last"),
    (40003, 70, 3001, np.float64, "blocks")])
def test_sorted_slices_bit_exact(ms, orc, d, n, k, dt, hmap):
    print("sorted slices d=%d n=%d k=%d %s %s" % (d, n, k, dt.__name__, hmap), flush=True)
    A = synth.normal_matrix(d, n, seed=d + k, dtype=dt)
    h = {"uniform": lambda: synth.bucket_map(d, k, seed=d),
         "one": lambda: np.full(d, k // 2, dtype=np.int32),
         "last": lambda: np.full(d, k - 1, dtype=np.int32),
         "blocks": lambda: (np.arange(d) // 700 % k).astype(np.int32)}[hmap]()
    s = synth.signs(d, seed=d + 1)
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(s), k, mode="sorted")
    ms.check_status(ws)
    assert bits_equal(to_host(Y), np.asfortranarray(orc.countsketch(A, h, s, k)))


# Uneven blocks of the same fold (one slice much longer than the others of its 4096
# rows), which keep full keys: none, one, some in a row with even ones between, fewer and more even
# ones than it takes to go back, all, the first and the last (not whole) block, and blocks whose
# long bucket comes first, last and at the middle key; two slices per thread, 1, 2 and 4 buckets
# a slice, and invalid rows beside them.  Bit-exact.
@pytest.mark.parametrize("pattern", ["u", "uu", "eu", "ue", "eeu", "ueeeu", "eeeeeu", "ueeeeeeeee",
                                     "ueeeeeeeeeue", "euueeuuue"])
@pytest.mark.parametrize("n,k,dt", [(2, 40, np.float64), (3, 4096, np.float32),
                                    (2, 8192, np.float64), (65, 16384, np.float64),
                                    (67, 9000, np.float32)])
def test_sorted_uneven_blocks(ms, orc, pattern, n, k, dt):
    d = 4096 * (len(pattern) - 1) + (4096 if len(pattern) % 2 else 1234)
    d = max(d, 4096)
    print("uneven blocks %s n=%d k=%d %s" % (pattern, n, k, dt.__name__), flush=True)
    A = synth.normal_matrix(d, n, seed=d + k, dtype=dt)
    h = synth.bucket_map(d, k, seed=k)
    rng = np.random.default_rng(len(pattern))
    for b, c in enumerate(pattern):
        if c == "u":
            rows = np.arange(4096 * b, min(d, 4096 * (b + 1)))
            # from 300 rows to all of them in one bucket
            pick = rng.random(rows.size) < (0.08, 0.5, 1.0)[b % 3]
            h[rows[pick]] = (0, k // 2, k - 1)[(b + n) % 3]
    s = synth.signs(d, seed=d + 1)
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(s), k, mode="sorted")
    ms.check_status(ws)
    assert bits_equal(to_host(Y), np.asfortranarray(orc.countsketch(A, h, s, k)))


# One workspace, its old contents all ones, for an even, an uneven and again an even map: what
# a call finds out about its blocks is not left to the next one.  Bit-exact.
def test_sorted_uneven_workspace_again(ms, orc):
    d, n, k = 20000, 9, 8192
    print("uneven workspace again", flush=True)
    A, s = synth.normal_matrix(d, n, seed=5), synth.signs(d, seed=6)
    h = synth.bucket_map(d, k, seed=7)
    u = h.copy()
    u[9000:9900] = 77
    ws = ms.workspace(ms.workspace_size("countsketch", d=d, n=n, k=k, mode="sorted"))
    ws.fill_(255)
    for hh in (h, u, h, u):
        Y, _ = ms.countsketch_apply(to_dev(A), to_dev(hh), to_dev(s), k, mode="sorted", ws=ws)
        ms.check_status(ws)
        assert bits_equal(to_host(Y), np.asfortranarray(orc.countsketch(A, hh, s, k)))


# Two slices a thread: the row counts around which they are taken (16,384 for two
# buckets a slice, 49,152 for four), beside one slice at the same sizes.  Bit-exact.
@pytest.mark.parametrize("d", [16383, 16384, 49151, 49152])
@pytest.mark.parametrize("n,k", [(66, 8192), (66, 16384), (9, 16384)])
def test_sorted_two_slices_rows(ms, orc, d, n, k):
    print("two slices d=%d n=%d k=%d" % (d, n, k), flush=True)
    A = synth.normal_matrix(d, n, seed=d + k)
    h, s = synth.bucket_map(d, k, seed=d), synth.signs(d, seed=d + 1)
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(s), k, mode="sorted")
    ms.check_status(ws)
    assert bits_equal(to_host(Y), np.asfortranarray(orc.countsketch(A, h, s, k)))


# FP32: from 4096 rows for two buckets a slice, 12,288 for four.  Bit-exact.
@pytest.mark.parametrize("d", [4096, 12287, 12288])
@pytest.mark.parametrize("n,k", [(66, 8192), (66, 16384), (128, 10000)])
def test_sorted_two_slices_rows_f32(ms, orc, d, n, k):
    print("two slices f32 d=%d n=%d k=%d" % (d, n, k), flush=True)
    A = synth.normal_matrix(d, n, seed=d + k, dtype=np.float32)
    h, s = synth.bucket_map(d, k, seed=d), synth.signs(d, seed=d + 1)
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(s), k, mode="sorted")
    ms.check_status(ws)
    assert bits_equal(to_host(Y), np.asfortranarray(orc.countsketch(A, h, s, k)))


def test_sorted_slices_special_values(ms, orc):
    # infinities, NaN, signed zeros and the smallest subnormal keep their bits
    # (a thread adds +0.0 to the sums of its other buckets)
    d, n, k = 9000, 3, 6000
    A = synth.normal_matrix(d, n, seed=2)
    A[::7] = -0.0
    A[5::97, 0] = np.inf
    A[11::501, 1] = -np.inf
    A[3::1009, 2] = 5e-324
    h, s = synth.bucket_map(d, k, seed=3), synth.signs(d, seed=4)
    Y, ws = ms.countsketch_apply(to_dev(A), to_dev(h), to_dev(s), k, mode="sorted")
    ms.check_status(ws)
    Yg, Yr = to_host(Y), np.asfortranarray(orc.countsketch(A, h, s, k))
    assert np.array_equal(np.isnan(Yg), np.isnan(Yr))
    ok = ~np.isnan(Yr)
    assert bits_equal(Yg[ok], Yr[ok])
