"""Workspaces smaller than ms_workspace_size() gives now.

The query of the FP64 product (258 columns and more), of the wide normal
equations and of rand_cholQR once gave less: their partial sums covered fewer
workgroups.  A buffer of that size still serves (fewer workgroups, the same
results up to the order of sums), nothing is written past its end, and half of
it is refused.

Bar: both runs are within the 1e-12 normwise bar that each operation has
against the oracle for kappa(A) <= 10 (here about 1.3), so within 2e-12 of
each other.
"""
import pytest
import torch

from gpu_util import rel, to_host

pytestmark = pytest.mark.gpu

# op, d, n, nrhs, k, k2, FP32 data, FP32 G, the bytes that were enough
CASES = [("normal_equations", 131075, 256, 1, 0, 0, False, False, 14797312),
         ("normal_equations", 40001, 65, 13, 0, 0, True, False, 2099712),
         ("rand_cholqr", 20001, 128, 2, 1024, 256, False, False, 28774144),
         ("rand_cholqr", 31693, 200, 1, 1600, 400, True, True, 69941760),
         ("lstsq", 9072, 128, 13, 40000, 1024, False, False, 434888960),
         ("gaussian", 0, 258, 0, 16384, 1024, False, False, 27476224),
         ("multisketch", 50003, 258, 0, 16384, 1024, False, False, 61492992)]


@pytest.fixture(scope="module")
def ms():
    import paper_2508_14209_amd as ms
    return ms


@pytest.mark.parametrize("op,d,n,nrhs,k,k2,f32,g32,old", CASES)
def test_smaller_workspace(ms, op, d, n, nrhs, k, k2, f32, g32, old):
    print("%s d=%d n=%d nrhs=%d k=%d k2=%d" % (op, d, n, nrhs, k, k2), flush=True)
    dt, gt = torch.float32 if f32 else torch.float64, torch.float32 if g32 else torch.float64
    gen = torch.Generator("cuda").manual_seed(d + n)

    def cm(r, c, t):
        return torch.randn(c, r, generator=gen, dtype=t, device="cuda").t()

    A = cm(d if op != "gaussian" else k, n, dt)
    if nrhs:
        B = (A.double() @ cm(n, nrhs, torch.float64) + 0.01 * cm(d, nrhs, torch.float64))
        B = B.to(dt).t().contiguous().t()
    if k:
        G = cm(k2, k, gt) * k2 ** -0.5
        G = G.t().contiguous().t()
        h = torch.randint(0, k, (max(d, 1),), generator=gen, device="cuda", dtype=torch.int32)
        s = (torch.randint(0, 2, (max(d, 1),), generator=gen, device="cuda") * 2 - 1).to(torch.int8)

    def run(ws):
        if op == "normal_equations":
            out = ms.normal_equations_lstsq(A, B, ws=ws)
        elif op == "rand_cholqr":
            out = ms.rand_cholqr_lstsq(A, B, h, s, G, k, ws=ws)
        elif op == "lstsq":
            out = ms.sketch_lstsq(A, B, h, s, G, k, ws=ws)
        elif op == "gaussian":
            out = ms.gaussian_apply(G, A, ws=ws)
        else:
            out = ms.multisketch_apply(A, h, s, G, k, ws=ws)
        ms.check_status(out[-1])
        return to_host(out[0])

    want = run(None)
    buf = torch.full((old + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    assert buf.data_ptr() % 256 == 0
    got = run(buf[:old])
    assert bool((buf[old:] == 0xA5).all())
    assert rel(got, want) <= 2e-12
    with pytest.raises(ms.MsketchError) as e:
        run(buf[:old // 2])
    assert e.value.code == ms.MS_ERR_NOMEM
