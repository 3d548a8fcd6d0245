"""Times of calls that differ in one property, on the GPU: a shape, a row count or a
bucket map that is served by a rule of its own must not cost far more than its
neighbour.  Every bar is on the ratio of two times of the same process, well
above what was measured and well below what the fault that it guards against
cost.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ms():
    import paper_2508_14209_amd as ms
    return ms


def _us(fn, reps=12):
    """Least time of a call on the GPU, in microseconds."""
    fn()
    torch.cuda.synchronize()
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
          for _ in range(reps)]
    for a, b in ev:
        a.record()
        fn()
        b.record()
    torch.cuda.synchronize()
    return 1e3 * min(a.elapsed_time(b) for a, b in ev)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(rows, cols, dtype=torch.float64, seed=0):
    return torch.randn((cols, rows), generator=_gen(seed), device="cuda", dtype=dtype).t()


def _gaussian(ms, k2, k, n):
    G, Y = _normal(k2, k), _normal(k, n, seed=1)
    Z = ms.empty_colmajor(k2, n, torch.float64)
    ws = ms.workspace(ms.workspace_size("gaussian", n=n, k=k, k2=k2))
    us = _us(lambda: ms.gaussian_apply(G, Y, Z=Z, ws=ws))
    print("gaussian k2=%d k=%d n=%d: %.1f us" % (k2, k, n, us), flush=True)
    return us


# FP64 product: two column tiles fill the chip evenly, three do not divide it (1.17 times
# the columns took 2.1 times the time when a die got whole splits only).
def test_gaussian_f64_three_tiles(ms):
    assert _gaussian(ms, 16, 131072, 300) <= 1.6 * _gaussian(ms, 16, 131072, 257)


# ... and one split of many tiles has the whole chip too: no more than eight copies of the result
# (it takes 4.4; on one die alone it took 13.7).
def test_gaussian_f64_one_split(ms):
    src, dst = _normal(4096, 2000), ms.empty_colmajor(4096, 2000, torch.float64)
    copy = _us(lambda: dst.copy_(src))
    print("copy: %.1f us" % copy, flush=True)
    assert _gaussian(ms, 4096, 16, 2000) <= 8 * copy


# ... and one row costs no more than two (2.2 times when its slabs were all guarded).
def test_gaussian_f64_one_row(ms):
    assert _gaussian(ms, 1, 131072, 500) <= 1.5 * _gaussian(ms, 2, 131072, 500)


def _lstsq(ms, d, n, nrhs, k, k2, dtype, refine, mode="auto"):
    A, B = _normal(d, n, dtype), _normal(d, nrhs, dtype, seed=1)
    h = torch.randint(0, k, (d,), generator=_gen(2), dtype=torch.int32, device="cuda")
    s = torch.randint(0, 2, (d,), generator=_gen(3), dtype=torch.int8, device="cuda") * 2 - 1
    G = _normal(k2, k, dtype, seed=4)
    X = ms.empty_colmajor(n, nrhs, torch.float64)
    dt = ms.MS_F64 if dtype == torch.float64 else ms.MS_F32
    ws = ms.workspace(ms.workspace_size("lstsq", d=d, n=n, nrhs=nrhs, k=k, k2=k2, a_dtype=dt,
                                        g_dtype=dt, mode=mode, refine_steps=refine))
    us = _us(lambda: ms.sketch_lstsq(A, B, h, s, G, k, mode=mode, refine_steps=refine, X=X, ws=ws))
    print("lstsq d=%d n=%d nrhs=%d refine=%d: %.1f us" % (d, n, nrhs, refine, us), flush=True)
    return us


# The last one to three rows of a refinement's residual: a row count that is no multiple of
# four costs what its neighbour costs (1.6 to 2.1 times when they were one lane's chain).
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_refinement_odd_rows(ms, dtype):
    args = (256, 8, 1024, 256, dtype, 8)
    assert _lstsq(ms, 100003, *args) <= 1.25 * _lstsq(ms, 100000, *args)


# ... also one row past whole workgroups of the widest kind (7 % of eight steps when its
# loads went past the caches and one after another).
def test_refinement_one_row_more(ms):
    args = (256, 1, 1024, 256, torch.float64, 8)
    assert _lstsq(ms, 4194305, *args) <= 1.06 * _lstsq(ms, 4194304, *args)


# 2.5 % more rows than one round of the widest workgroups: a second, nearly empty round took half as
# long again.
def test_refinement_nearly_empty_round(ms):
    args = (64, 1, 256, 64, torch.float64, 8)
    assert _lstsq(ms, 4300000, *args) <= 1.2 * _lstsq(ms, 4194304, *args)


# The deterministic CountSketch with 64 rows in a row to a bucket: a block's longest chain is 64
# adds, four times the time of even buckets at most (seven times when four buckets' chains were
# one thread's).
def test_sorted_uneven_buckets(ms):
    d, n, k = 1000003, 65, 16384
    A, Y = _normal(d, n), ms.empty_colmajor(k, n, torch.float64)
    s = torch.randint(0, 2, (d,), generator=_gen(3), dtype=torch.int8, device="cuda") * 2 - 1
    ws = ms.workspace(ms.workspace_size("countsketch", d=d, n=n, k=k, mode="sorted"))
    even = torch.randint(0, k, (d,), generator=_gen(2), dtype=torch.int32, device="cuda")
    runs = ((torch.arange(d, device="cuda") // 64) % k).int()
    a, b = (_us(lambda: ms.countsketch_apply(A, h, s, k, Y=Y, ws=ws, mode="sorted"))
            for h in (even, runs))
    print("even %.1f us, runs %.1f us" % (a, b), flush=True)
    assert b <= 4 * a


# Two bucket tiles over data that the caches hold: one column more than three for each of a die's
# groups costs no more than an even share (a quarter more when the left-over column's pieces were
# flushed all at one time).
def test_two_tiles_left_over_column(ms):
    def us(n):
        d, k = 1000000, 32768
        A, Y = _normal(d, n, torch.float32), ms.empty_colmajor(k, n, torch.float32)
        h = torch.randint(0, k, (d,), generator=_gen(2), dtype=torch.int32, device="cuda")
        s = torch.randint(0, 2, (d,), generator=_gen(3), dtype=torch.int8, device="cuda") * 2 - 1
        ws = ms.workspace(ms.workspace_size("countsketch", d=d, n=n, k=k, a_dtype=ms.MS_F32))
        t = _us(lambda: ms.countsketch_apply(A, h, s, k, Y=Y, ws=ws), 24)
        print("n=%d: %.1f us" % (n, t), flush=True)
        return t

    assert us(49) <= 1.12 * us(48)
