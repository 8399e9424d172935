"""The particle sort at the edges of its plans: blocks of 1024 and 4096 keys
and their remainders, the largest sort without a scan (256 blocks) and the
next, digits of 8 and 9 bits, one to three passes, the allocation-free entry
point; against a stable library sort, exactly."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _ctx(ncell):
    from paper_1908_10793_amd import dust
    faces = [np.linspace(0.0, 1.0, ncell[d] + 1) for d in range(3)]
    box = dict(geom="cart", ndim=3, n=ncell, bc_lo=("periodic",) * 3, bc_hi=("periodic",) * 3, shape=("cic",) * 3,
               faces=faces)
    return dust.Context([box], prec="f32")


# cells: 8 bits (255 bins and the one of the cell-less: 256 keys), 9, 17, 18, 19 and 20 bits
CELLS = [(5, 3, 17), (16, 16, 1), (64, 32, 32), (64, 64, 63), (64, 64, 64), (128, 64, 64)]


@pytest.mark.parametrize("n", [1, 1023, 1025, 256 * 1024 - 1, 256 * 1024, 256 * 1024 + 1, (1 << 19) - 1, 1 << 19,
                               (1 << 19) + 4097])
@pytest.mark.parametrize("cells", CELLS)
def test_sort_is_the_stable_sort(cells, n):
    ctx = _ctx(cells)
    C = int(np.prod(cells))
    rng = np.random.default_rng(n)
    for kind in ("random", "sorted", "one"):
        c = rng.integers(-1, C, size=n).astype(np.int32)
        if kind == "sorted":
            c.sort()
        elif kind == "one":
            c[:] = C - 1
        t = torch.from_numpy(c).cuda()
        P = {"cell": t, "off": [torch.zeros(n, device="cuda")] * 3, "mom": [torch.zeros(n, device="cuda")] * 3}
        ref_perm, ref_start = O.bin_reference(c.astype(np.int64), C)
        for call in (ctx.bin, ctx.bin_noalloc):
            perm = torch.full((n,), -7, dtype=torch.int32, device="cuda")
            start = torch.full((C + 1,), -7, dtype=torch.int64, device="cuda")
            call(P, perm=perm, bin_start=start)
            assert np.array_equal(perm.cpu().numpy(), ref_perm), (kind, call.__name__)
            assert np.array_equal(start.cpu().numpy(), ref_start), (kind, call.__name__)
