"""K5's tile sizes (256, and 128 or 64 where 256 tiles would leave compute
units idle): the same problem through each of them gives the same bits, and
those lie within the oracle's bound.  The tile of a launch follows from its
problems, so a problem gets the 256 tile in a batch with a large filler and
the 128 tile with a medium one."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import require_gpu
from oracle import wgrad as W
from synth import wgrad as SW

pytestmark = pytest.mark.gpu

SS_RTOL = 264 * 2.0 ** -24


def to_dev(torch, bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to("cuda")


def launch(torch, problems, filler):
    """dw and tile sums of the problems (dy, x, old dw, accumulate), batched
    with a filler problem of filler x filler features and 320 tokens when
    filler > 0."""
    from paper_2606_00539_amd import gnmr_wgrad_num_tiles, gnmr_wgrad_sumsq_batched

    probs = [(to_dev(torch, dy), to_dev(torch, x), to_dev(torch, old), dy.shape[0], dy.shape[1],
              x.shape[1], acc) for dy, x, old, acc in problems]
    if filler:
        z = torch.zeros((320, filler), dtype=torch.int16, device="cuda")
        for acc in sorted({p[6] for p in probs}):
            out = torch.zeros((filler, filler), dtype=torch.int16, device="cuda")
            probs.append((z, z, out, 320, filler, filler, acc))
    off = np.concatenate([[0], np.cumsum([gnmr_wgrad_num_tiles(p[4], p[5]) for p in probs])])
    ss = torch.full((int(off[-1]),), float("nan"), dtype=torch.float32, device="cuda")
    gnmr_wgrad_sumsq_batched(probs, ss)
    torch.cuda.synchronize()
    ss = ss.cpu().numpy()
    return [(p[2].cpu().numpy().view(np.uint16), ss[off[i]:off[i + 1]])
            for i, p in enumerate(probs[:len(problems)])]


# tile edges of 64, 128 and 256 and one vector past them; tokens around the K
# step of 64 and the staging rings of two and four steps
@pytest.mark.parametrize("M,N,T", [(8, 8, 256), (64, 72, 257), (72, 64, 319), (128, 136, 320),
                                   (136, 264, 321), (256, 328, 449), (264, 520, 512),
                                   (520, 248, 577), (1160, 1096, 1025)])
def test_every_tile_size_gives_the_same_bits(M, N, T):
    torch = require_gpu()
    print(f"wgrad tiles M={M} N={N} T={T}", flush=True)
    dy, x = SW.operands(3, 1, M + N, tokens=T, out_f=M, in_f=N)
    old = W.bf16_rne(np.random.default_rng(M * N).standard_normal((M, N)) * 0.02)
    problems = [(dy, x, old, 0), (dy, x, old, 1)]
    small = launch(torch, problems, 0)          # 64: at most 256 workgroups, 512 from 1,024 tokens
    medium = launch(torch, problems, 1280)      # 128: over 256 of 64, under 256 of 128
    large = launch(torch, problems, 3072)       # 256
    for (acc, a, b, c) in zip((0, 1), small, medium, large):
        for name, other in (("128", b), ("256", c)):
            assert np.array_equal(a[0], other[0]), f"accumulate={acc}: dw of the {name} tile"
            assert np.array_equal(a[1], other[1]), f"accumulate={acc}: sums of the {name} tile"
        if acc:
            exact = W.wgrad_accumulate_exact(old, dy, x)
            bound = W.error_bound_accumulate(old, dy, x, exact)
        else:
            exact = W.wgrad_exact(dy, x)
            bound = W.error_bound(dy, x, exact)
        assert np.all(np.abs(W.widen_bf16(a[0]) - exact) <= bound), f"accumulate={acc}"
        np.testing.assert_allclose(a[1], W.tile_sumsq(a[0]), rtol=SS_RTOL, atol=0)


# rows a multiple of 4,096 bytes apart, in 64, 128 and 256 tiles with ragged edges
@pytest.mark.parametrize("M,N,T", [(264, 2048, 300), (776, 2048, 700), (2056, 4096, 64)])
def test_accumulated_tiles_stored_in_rows(M, N, T):
    """Alone, most tiles of the launch have such rows and are stored row by row;
    with a filler whose rows are 6,144 bytes apart they are stored directly."""
    torch = require_gpu()
    print(f"wgrad rows M={M} N={N} T={T}", flush=True)
    dy, x = SW.operands(5, 1, M + N, tokens=T, out_f=M, in_f=N)
    old = W.bf16_rne(np.random.default_rng(M).standard_normal((M, N)) * 0.02)
    (rows, ss), = launch(torch, [(dy, x, old, 1)], 0)
    (direct, ss_direct), = launch(torch, [(dy, x, old, 1)], 3072)
    assert np.array_equal(rows, direct) and np.array_equal(ss, ss_direct)
    exact = W.wgrad_accumulate_exact(old, dy, x)
    assert np.all(np.abs(W.widen_bf16(rows) - exact) <= W.error_bound_accumulate(old, dy, x, exact))
    np.testing.assert_allclose(ss, W.tile_sumsq(rows), rtol=SS_RTOL, atol=0)


def test_more_problems_than_one_launch_holds():
    """35 problems (a launch holds 32) of differing sizes and both kinds: every
    dw the oracle's bit for bit on integer operands, tile sums at the
    concatenated offsets."""
    torch = require_gpu()
    shapes = [(8 * (1 + i % 5), 8 * (1 + i % 7), 40 + i) for i in range(35)]
    problems = []
    for i, (M, N, T) in enumerate(shapes):
        dy, x = SW.small_integer_operands(50 + i, T, M, N)
        old = W.bf16_rne(np.random.default_rng(i).integers(-8, 9, (M, N)).astype(np.float64))
        problems.append((dy, x, old, i % 2))
    for i, ((dy, x, old, acc), (dw, ss)) in enumerate(zip(problems, launch(torch, problems, 0))):
        want = W.bf16_rne(W.wgrad_accumulate_exact(old, dy, x) if acc else W.wgrad_exact(dy, x))
        assert np.array_equal(dw, want), f"problem {i}"
        np.testing.assert_allclose(ss, W.tile_sumsq(want), rtol=SS_RTOL, atol=0,
                                   err_msg=f"problem {i}")


# Around the limits at which the tile of one problem changes: 256 and 512 tiles of 64
# and of 128, steps that do and do not pay, problems no higher or wider than a tile.
# The 256 tile beside a filler gives the same bits.
@pytest.mark.parametrize("M,N,T", [
    (1024, 1024, 255), (1024, 1032, 256), (1408, 1472, 1023), (1408, 1472, 960),
    (64, 16392, 1024), (72, 16392, 1024), (2048, 2048, 448), (2048, 2048, 449),
    (2056, 2048, 1984), (2816, 2816, 1985), (128, 38400, 2048), (128, 50000, 2048),
    (136, 32776, 2048), (38400, 8, 2048)])
def test_one_problem_where_its_tile_changes(M, N, T):
    torch = require_gpu()
    print(f"wgrad tile rule M={M} N={N} T={T}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N + T)
    bits = lambda *shape: torch.randn(shape, generator=g, device="cuda").bfloat16().view(
        torch.int16).cpu().numpy()
    dy, x = bits(T, M), bits(T, N)
    (dw, ss), = launch(torch, [(dy, x, np.zeros((M, N), np.int16), 0)], 0)
    (want, ss_want), = launch(torch, [(dy, x, np.zeros((M, N), np.int16), 0)], 5888)
    assert np.array_equal(dw, want) and np.array_equal(ss, ss_want)
