"""A small workload's step in one launch gives the bits of the step whose kernels
are launched one by one (which profiling asks for), up to and past its limits."""
import numpy as np
import pytest

from gpu_util import require_gpu
from paper_2606_00539_amd import GNMR_BF16, GNMR_F32, Controller

pytestmark = pytest.mark.gpu
ITEM = 65536  # bytes
FIELDS = ("mask", "lock", "norm", "gnmr", "dgnmr", "risk")


def sizes_of(units, items, dtype):
    """Values per unit: `items` work items in all, shared as evenly as they go,
    the last of each unit ragged (an empty unit where a share is 0)."""
    per = ITEM // (2 if dtype == GNMR_BF16 else 4)
    share = [items // units + (b < items % units) for b in range(units)]
    return [n * per - (37 * b + 5) % 1000 if n else 0 for b, n in enumerate(share)]


# (units, items): one lane, a wavefront or a workgroup's order per unit; around
# 1,024 items (the late ones), 256 units and 6,144 items
@pytest.mark.parametrize("units,items,dtype", [
    (1, 1, GNMR_F32), (1, 33, GNMR_BF16), (28, 196, GNMR_F32), (3, 1023, GNMR_BF16),
    (30, 1024, GNMR_BF16), (33, 1057, GNMR_BF16), (84, 6048, GNMR_BF16), (256, 100, GNMR_F32),
    (256, 6144, GNMR_BF16), (192, 6144, GNMR_BF16), (7, 6144, GNMR_BF16), (1, 6144, GNMR_BF16),
    (257, 300, GNMR_F32), (100, 6145, GNMR_BF16)])
@pytest.mark.parametrize("passed", [False, True])
def test_one_launch_gives_the_bits_of_several(units, items, dtype, passed):
    torch = require_gpu()
    print("one launch", units, items, dtype, passed, flush=True)
    sizes = sizes_of(units, items, dtype)
    g = torch.Generator(device="cuda").manual_seed(units * 10007 + items)
    flat = torch.empty(sum(sizes) + 8 * units, device="cuda",
                       dtype=torch.bfloat16 if dtype == GNMR_BF16 else torch.float32)
    segs, at = [], 0
    for b, n in enumerate(sizes):   # addresses that are not multiples of 16
        segs.append(flat[at:at + n])
        at += n + b % 8
    off = np.arange(units + 1)
    cfg = dict(window=3, max_o=max(1, units // 8), lock_len=2, eps=1e-12)
    args = (off, sizes, [dtype] * units, None if passed else segs)
    rng = np.random.default_rng(units + items)
    with Controller(units, *cfg.values(), *args) as one, \
            Controller(units, *cfg.values(), *args) as ref:
        assert one.info()["num_items"] == items
        ref.set_profiling(True)
        for t in range(1, 7):
            flat.normal_(0.0, 1e-3, generator=g)
            for b in rng.choice(units, max(1, units // 4), replace=False):
                segs[b].mul_(float(rng.uniform(2, 20)))
            if t == 5:
                segs[0].fill_(float("inf"))
            for c in (one, ref):
                c.step(1.1, 1.3, seg_ptr=segs if passed else None)
            a, b = one.query(), ref.query()
            for k in FIELDS:
                assert a[k].tobytes() == b[k].tobytes(), (t, k)
            assert a["stats"] == b["stats"] and a["stats"]["t"] == t
            if t == 3:   # a state taken back: the same step number again
                saved = one.get_state()
            if t == 4:
                one.set_state(saved)
                ref.set_state(saved)
                for c in (one, ref):
                    c.step(1.1, 1.3, seg_ptr=segs if passed else None)
                a, b = one.query(), ref.query()
                assert all(a[k].tobytes() == b[k].tobytes() for k in FIELDS)
                assert a["stats"]["t"] == 4


def uneven(counts, dtype, empty):
    """CSR offsets and segment sizes of units of counts[b] work items, in up to two
    segments; a unit of none has no segment, or (`empty`) two of no values."""
    per = ITEM // (2 if dtype == GNMR_BF16 else 4)
    off, sizes = [0], []
    for b, n in enumerate(counts):
        if n > 1:
            sizes += [(n // 2) * per, (n - n // 2) * per - 3 * b - 1]
        elif n or empty:
            sizes += [per - 1] if n else [0, 0]
        off.append(len(sizes))
    return np.array(off, np.int64), sizes


# Units without items first, in the middle and last, and units of very different
# sizes: a wavefront's and a workgroup's order per unit, below, at and above the
# 1,024 items that are all collected at once.
@pytest.mark.parametrize("counts", [
    [100, 0], [64, 0], [0, 400, 400], [40, 0, 100, 50], [1023, 0], [1024, 0], [1025, 0],
    [512, 0, 512], [513, 0, 512], [2000, 0, 2000], [0] + [40] * 20, [40] * 10 + [0] + [40] * 10,
    [40] * 20 + [0], [0, 0, 300, 0], [3, 900, 1, 100], [1, 2500, 0, 2, 1200, 60, 2],
    [0] + [60, 3, 200, 0] * 12], ids=lambda c: f"{len(c)}u{sum(c)}i{c.index(0) if 0 in c else ''}")
@pytest.mark.parametrize("empty", [False, True])
@pytest.mark.parametrize("passed", [False, True])
def test_units_without_items_and_uneven_units(counts, empty, passed):
    torch = require_gpu()
    from paper_2606_00539_amd import gnmr_wgrad_num_tiles, gnmr_wgrad_sumsq

    print("uneven units", counts, empty, passed, flush=True)
    U, none = len(counts), np.array(counts) == 0
    off, sizes = uneven(counts, GNMR_BF16, empty)
    g = torch.Generator(device="cuda").manual_seed(sum(counts))
    flat = torch.empty(sum(sizes), device="cuda", dtype=torch.bfloat16)
    segs, at = [], 0
    for n in sizes:
        segs.append(flat[at:at + n] if n else 0)
        at += n
    args = (off, sizes, [GNMR_BF16] * len(sizes), None if passed else segs)
    # other kernels leave their operands in the compute units' LDS
    dy = torch.randn(64, 4096, device="cuda", generator=g).bfloat16() + 3
    dw = torch.empty(4096, 4096, device="cuda", dtype=torch.bfloat16)
    sums = torch.empty(gnmr_wgrad_num_tiles(4096, 4096), device="cuda")
    with Controller(U, 3, 1, 2, 1e-12, *args) as one, \
            Controller(U, 3, 1, 2, 1e-12, *args) as ref:
        assert one.info()["num_items"] == sum(counts)
        ref.set_profiling(True)
        for t in range(1, 6):
            flat.normal_(0.0, 1e-3 * t, generator=g)
            gnmr_wgrad_sumsq(dy, dy, dw, 64, 4096, 4096, sums)
            for c in (one, ref):
                c.step(1.1, 1.3, seg_ptr=segs if passed else None)
            a, b = one.query(), ref.query()
            assert np.all(a["norm"][none] == 0.0), (t, a["norm"][none])
            for k in FIELDS:
                assert a[k].tobytes() == b[k].tobytes(), (t, k)
            assert a["stats"] == b["stats"]
