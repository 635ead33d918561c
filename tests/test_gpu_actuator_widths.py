"""K4's row classes: each width class's edges, rows of several units in one
wavefront, and both kinds of loads, against the oracle bit for bit."""
import numpy as np
import pytest

from gpu_util import require_gpu
from oracle import fakequant as FQ

pytestmark = pytest.mark.gpu

# the widest row of every class and one vector more
WIDTHS = [8] + [w + d for w in (128, 256, 512, 1024, 1536, 2048, 3072, 4096, 6144, 8192, 12288)
                for d in (0, 8)] + [16384]
LOW, REC = 1, 0      # E2M1, BF16


def rows_of(rng, rows, cols):
    x = rng.normal(size=(rows, cols)).astype(np.float32) * (10.0 ** rng.uniform(-6, 2, (rows, 1)))
    x[rows // 2] = 0.0
    return FQ.f32_to_bf16(x.astype(np.float32))


def to_device(torch, a):
    return torch.from_numpy(a.view(np.int16).copy()).to("cuda")


@pytest.mark.parametrize("fmts", [(LOW, REC), (5, 3)])
@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("large", [False, True])
def test_every_width_class_from_the_table(fmts, inplace, large):
    """Two segments per width (3 and 8 rows, neighbouring units, so that short
    rows of both paths share wavefronts).  `large`: a further segment of 69 MB
    makes the set too big for cached loads; its unit recovers in BF16 in
    place, or it has no rows to check otherwise."""
    torch = require_gpu()
    from paper_2606_00539_amd import Actuator

    print(f"actuator widths fmts={fmts} inplace={inplace} large={large}", flush=True)
    rng = np.random.default_rng(sum(fmts) + 2 * inplace)
    acts = [rows_of(rng, r, c) for c in WIDTHS for r in (3, 8)]
    U = len(acts) + 1
    mask = (np.arange(U) % 2).astype(np.uint8)
    mask[-1] = 1
    d_in = [to_device(torch, a) for a in acts]
    d_out = d_in if inplace else [torch.full_like(t, 0x5555) for t in d_in]
    segs = [(i, o, a.shape[0], a.shape[1], b)
            for b, (i, o, a) in enumerate(zip(d_in, d_out, acts))]
    if large:
        big = torch.zeros((2100, 16384), dtype=torch.int16, device="cuda")
        segs.append((big, big, 2100, 16384, U - 1))
    with Actuator(segs, U) as act:
        act.apply(torch.from_numpy(mask).to("cuda"), *fmts)
        torch.cuda.synchronize()
    for b, (o, w) in enumerate(zip(d_out, FQ.actuate(acts, mask[:-1], *fmts))):
        got = o.cpu().numpy().view(np.uint16).reshape(w.shape)
        assert np.array_equal(got, w), f"cols {w.shape[1]} rows {w.shape[0]} mask {mask[b]}"


@pytest.mark.parametrize("cols", WIDTHS)
def test_every_width_class_as_a_matrix(cols):
    torch = require_gpu()
    from paper_2606_00539_amd import gnmr_actuate_matrix

    print(f"actuator matrix cols={cols}", flush=True)
    x = rows_of(np.random.default_rng(cols), 13, cols)
    d = to_device(torch, x)
    mask = torch.tensor([0, 1], dtype=torch.uint8, device="cuda")
    for unit, fmt in ((0, LOW), (1, 3)):
        out = torch.full((14, cols), 0x5555, dtype=torch.int16, device="cuda")
        gnmr_actuate_matrix(d, out, 13, cols, mask, unit, LOW, 3)
        torch.cuda.synchronize()
        got = out.cpu().numpy().view(np.uint16)
        assert np.array_equal(got[:13], FQ.fakequant_rows(x, fmt))
        assert np.all(got[13] == 0x5555), "written past the last row"


@pytest.mark.parametrize("rows,cols", [(70000, 512), (17000, 2056), (2100, 16384)])
def test_large_matrix_equals_its_parts(rows, cols):
    """Past 64 MB the loads are non-temporal: the same rows as calls below it."""
    torch = require_gpu()
    from paper_2606_00539_amd import gnmr_actuate_matrix

    assert rows * cols * 2 > 64 << 20
    print(f"actuator large matrix {rows}x{cols}", flush=True)
    x = torch.randn(rows, cols, device="cuda").bfloat16()
    mask = torch.zeros(1, dtype=torch.uint8, device="cuda")
    whole, parts = torch.empty_like(x), torch.empty_like(x)
    gnmr_actuate_matrix(x, whole, rows, cols, mask, 0, LOW, REC)
    half = rows // 2
    gnmr_actuate_matrix(x[:half], parts[:half], half, cols, mask, 0, LOW, REC)
    gnmr_actuate_matrix(x[half:], parts[half:], rows - half, cols, mask, 0, LOW, REC)
    torch.cuda.synchronize()
    assert torch.equal(whole.view(torch.int16), parts.view(torch.int16))


# all classes in one launch, with ordinary loads up to 64 MB of input and
# non-temporal ones past it; rows that fill their class's workgroups and rows that
# do not
@pytest.mark.parametrize("rows", [1, 8, 33])
@pytest.mark.parametrize("widths", [(8, 136), (1024, 2312), (128, 3080, 16384), tuple(WIDTHS)])
@pytest.mark.parametrize("past", [0, 1])
def test_classes_of_a_small_table_in_one_launch(rows, widths, past):
    torch = require_gpu()
    from paper_2606_00539_amd import Actuator

    print(f"actuator mixed {rows} {widths} {past}", flush=True)
    rng = np.random.default_rng(rows + len(widths))
    acts = [rows_of(rng, rows, c) for c in widths]
    U = len(acts) + 1
    fill = ((64 << 20) - sum(a.size * 2 for a in acts)) // 2048 + past
    filler = torch.zeros((fill, 1024), dtype=torch.int16, device="cuda")
    mask = (np.arange(U) % 2).astype(np.uint8)
    d_in = [to_device(torch, a) for a in acts]
    d_out = [torch.full_like(t, 0x5555) for t in d_in]
    segs = [(i, o, rows, a.shape[1], b) for b, (i, o, a) in enumerate(zip(d_in, d_out, acts))]
    for few in (False, True):
        for o in d_out:
            o.fill_(0x5555)
        with Actuator(segs + ([] if few else [(filler, filler, fill, 1024, U - 1)]), U) as act:
            act.apply(torch.from_numpy(mask).to("cuda"), LOW, 3)
            torch.cuda.synchronize()
        for o, w in zip(d_out, FQ.actuate(acts, mask[:-1], LOW, 3)):
            got = o.cpu().numpy().view(np.uint16).reshape(w.shape)
            assert np.array_equal(got, w), f"cols {w.shape[1]}"
    assert not filler.any()


# a launch per class: past 384 MB, and past 64 MB where more than 32 MB for each
# class but one are rows of two vectors a lane; below either, one launch
@pytest.mark.parametrize("widths,filler,rows", [
    (tuple(WIDTHS), 16384, 12500), (tuple(WIDTHS), 16384, 11500),
    ((2312,), 1024, 34000), ((1000, 8192, 12296), 512, 100000), ((1000, 8192, 12296), 512, 70000),
    ((6144,), 2048, 17000)])
def test_classes_of_a_large_table(widths, filler, rows):
    torch = require_gpu()
    from paper_2606_00539_amd import Actuator

    print(f"actuator large table {len(widths)} widths, {rows} x {filler}", flush=True)
    rng = np.random.default_rng(rows)
    acts = [rows_of(rng, r, c) for c in widths for r in (3, 33)]
    U = len(acts) + 1
    mask = (np.arange(U) % 2).astype(np.uint8)
    mask[-1] = 0
    fill = torch.zeros((rows, filler), dtype=torch.int16, device="cuda")
    fill[rows - 1] = to_device(torch, rows_of(rng, 1, filler))[0]
    last = fill[rows - 1].cpu().numpy().view(np.uint16)[None]
    d_in = [to_device(torch, a) for a in acts]
    d_out = [torch.full_like(t, 0x5555) for t in d_in]
    segs = [(i, o, a.shape[0], a.shape[1], b)
            for b, (i, o, a) in enumerate(zip(d_in, d_out, acts))]
    with Actuator(segs + [(fill, fill, rows, filler, U - 1)], U) as act:
        act.apply(torch.from_numpy(mask).to("cuda"), LOW, 3)
        torch.cuda.synchronize()
    for o, w in zip(d_out, FQ.actuate(acts, mask[:-1], LOW, 3)):
        assert np.array_equal(o.cpu().numpy().view(np.uint16).reshape(w.shape), w), w.shape
    got = fill[rows - 1].cpu().numpy().view(np.uint16)[None]
    assert np.array_equal(got, FQ.fakequant_rows(last, LOW)) and not fill[:-1].any()


@pytest.mark.parametrize("cols", WIDTHS)
def test_a_table_of_one_width(cols):
    """A table of one class takes that class's own kernel."""
    torch = require_gpu()
    from paper_2606_00539_amd import Actuator

    print(f"actuator table of one width {cols}", flush=True)
    rng = np.random.default_rng(cols)
    acts = [rows_of(rng, r, cols) for r in (1, 3, 33)]
    mask = np.array([0, 1, 0], np.uint8)
    d_in = [to_device(torch, a) for a in acts]
    d_out = [torch.full_like(t, 0x5555) for t in d_in]
    segs = [(i, o, a.shape[0], cols, b) for b, (i, o, a) in enumerate(zip(d_in, d_out, acts))]
    with Actuator(segs, 3) as act:
        act.apply(torch.from_numpy(mask).to("cuda"), LOW, 3)
        torch.cuda.synchronize()
    for o, w in zip(d_out, FQ.actuate(acts, mask, LOW, 3)):
        assert np.array_equal(o.cpu().numpy().view(np.uint16).reshape(w.shape), w)
