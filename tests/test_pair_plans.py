"""Both residual blocks of a section in one launch: its strips on the CPU, its kernel against the oracle and the other kernels."""
import random

import numpy as np
import pytest

from paper_1910_06591_amd import workloads as wl
from tests import batch_bits, host_program

MAIN = r"""
// per map: LDS bytes, the most pixel tiles of a wavefront and its limit, pixels of the incoming map asked for and needed, and
// whether the strips cover every row once with their halos inside the map
int main()
{
    int H, W, C, B;
    while (scanf("%d %d %d %d", &H, &W, &C, &B) == 4) {
        strip_by_width(C, [&](auto cc) {
            constexpr int CC = decltype(cc)::value;
            using K = PairCfg<CC>;
            PairPlan p;
            if (!p.choose<CC>(H, W)) { printf("-\n"); return true; }
            const int stack = p.stack<CC>(B, H, W, 256), rows = p.rows(H, stack), pixels = p.pixels(H, W, stack);
            int need = stack > 1 ? stack * H * W : 0, most = stack > 1 ? stack * (H + 1) - 1 : 0, covered = 0;
            for (int s = 0; s < p.strips; ++s) {
                const int y0 = s * p.TH, ye = std::min(y0 + p.TH, H);
                covered += std::max(ye - y0, 0);
                if (stack > 1) continue;
                need = std::max(need, (std::min(ye + 4, H) - std::max(y0 - 4, 0)) * W);
                most = std::max(most, std::min(ye + 3, H) - std::max(y0 - 3, 0));
            }
            const int tiles = (K::S::tiles(rows, W) + K::S::NPG - 1) / K::S::NPG;
            printf("%zu %d %d %d %d %d\n", K::lds_bytes(rows, pixels, W), tiles, K::TPW, pixels, need, covered == H && most <= rows && (stack == 1 || p.strips == 1));
            return true;
        });
    }
}
"""


def test_strips_fit_lds_and_the_registers(tmp_path):
    """The map and the incoming pixels fit LDS, the pixel tiles the registers, and the rows of the launch those of its
    longest strip, for whole images, stacks and up to many strips."""
    rng = random.Random(3)
    maps = [(1, 1), (1, 300), (200, 1), (9, 12), (18, 24), (36, 48), (54, 72), (45, 60), (5, 3)]
    maps += [(rng.randint(1, 150), rng.randint(1, 250)) for _ in range(300)]
    cases = [(h, w, c, rng.choice([1, 300, 600, 1100, 2051])) for h, w in maps for c in (16, 32, 64, 128)]
    out = host_program.build(tmp_path, MAIN)([" ".join(map(str, c)) for c in cases])
    assert len(out) == len(cases)
    for case, line in zip(cases, out):
        if line != "-":
            lds, tiles, limit, pixels, need, cover = map(int, line.split())
            assert lds <= 160 * 1024 and 1 <= tiles <= limit and need <= pixels and cover, (case, line)
    assert sum(line != "-" for line in out) > len(out) // 2


def test_stacks_go_by_whole_rounds(tmp_path):
    """Images per workgroup on 256 compute units: one while a round holds the batch, then as many as keep the rounds few."""
    main = r"""
int main()
{
    int H, W, C, B;
    while (scanf("%d %d %d %d", &H, &W, &C, &B) == 4)
        strip_by_width(C, [&](auto cc) {
            PairPlan p;
            p.choose<decltype(cc)::value>(H, W);
            printf("%d\n", p.stack<decltype(cc)::value>(B, H, W, 256));
            return true;
        });
}
"""
    batches = (1, 256, 257, 511, 512, 513, 768, 769, 1000, 1024)
    want = {(9, 12, 16): (1, 1, 2, 2, 2, 3, 3, 4, 4, 4), (9, 12, 64): (1, 1, 2, 2, 2, 3, 3, 4, 4, 4),
            (18, 24, 32): (1, 1, 2, 2, 2, 1, 1, 2, 2, 2), (13, 13, 64): (1, 1, 2, 2, 2, 3, 3, 2, 2, 2),
            (18, 24, 64): (1,) * 10, (36, 48, 32): (1,) * 10}                # one fits; strips
    cases = [(*m, b) for m in want for b in batches]
    out = host_program.build(tmp_path, main)([" ".join(map(str, c)) for c in cases])
    assert dict(zip(cases, map(int, out))) == {(*m, b): s for m, stacks in want.items() for b, s in zip(batches, stacks)}


# frames, sections, rows; the kernels at that many rows and at one (first layer, then blocks)
CASES = [
    ((120, 192, 3), (16,), 300, "rows6 pair:4", "tile tile"),              # four strips, inner ones with halos on both sides
    ((119, 80, 4), (32,), 130, "rows12 pair:3", "tile tile"),
    ((59, 37, 3), (64,), 200, "tile pair:2", "tile tile"),                 # two strips of 15 rows
    ((36, 48, 3), (64,), 300, "rows9 pair*1", "tile tile"),                # whole images
    ((20, 100, 3), (32,), 301, "rows5 pair*2", "tile tile"),               # stacks, a last one of fewer images
    ((41, 67, 3), (16,), 601, "tile pair*3", "tile tile"),
    # (one map, one strip, one tile: the row alone is unstacked, on the same kernel)
    ((9, 13, 1), (16,), 1100, "tile pair*3", "tile pair*1"),               # feature rows padded to whole chunks
    ((9, 13, 16), (16, 32), 1025, "rows5 pair*3 pair*3", "tile pair*1 pair*1"),
]
# 128 channels run on strips at any batch where they can; behind 32 channels there are none for their conv0, so the blocks run
# on tiles: frames, rows, the kernels of sections (64, 128) and of (32, 128)
WIDE = [
    ((36, 48, 3), 256, "rows9 pair*1 pair*1", "tile pair*1 tile"),
    ((36, 48, 3), 301, "rows9 pair*1 pair*2", "tile pair*2 tile"),
    ((28, 40, 3), 601, "rows7 pair*1 pair*3", "rows14 pair*3 tile"),
    ((28, 28, 3), 1001, "rows7 pair*2 pair*4", "rows14 pair*4 tile"),
    ((64, 64, 3), 60, "tile tile pair*1", "tile tile tile"),
]


def test_cases_take_the_kernels_they_compare(tmp_path):
    out = batch_bits.routes(tmp_path, [(b, f, s) for f, s, rows, *_ in CASES for b in (rows, 1)])
    assert list(zip(out[::2], out[1::2])) == [(many, one) for *_, many, one in CASES]
    out = batch_bits.routes(tmp_path, [(rows, f, (c, 128)) for f, rows, *_ in WIDE for c in (64, 32)])
    assert list(zip(out[::2], out[1::2])) == [(wide, narrow) for *_, wide, narrow in WIDE]


@pytest.mark.gpu
@pytest.mark.parametrize("frame,sections,batch", [c[:3] for c in CASES], ids=str)
def test_one_launch_gives_the_bits_of_two(orc, frame, sections, batch):
    """Rows of a large batch, whose blocks run in one launch, equal the same rows in a batch of one, on the tile kernels
    where CASES says so, and the oracle."""
    batch_bits.check(orc, frame, sections, batch)


@pytest.mark.gpu
@pytest.mark.parametrize("frame,batch", [c[:2] for c in WIDE], ids=str)
def test_one_launch_gives_the_tile_kernels_bits_at_128_channels(frame, batch):
    """Sections (32, 128) on the tile kernels against (64, 128) with one launch for the second section's blocks, the same
    network: the upper 32 channels of the wide one's first section are zero all through (weights, biases), and so is what
    the second section takes from them; whole chunks of zeros add nothing to a sum."""
    h, w, c = frame
    cfg = {n: dict(wl.CONFIGS["C3"], label=f"{h}x{w}x{c}, sections {n} 128", index=132, obs_h=h, obs_w=w, obs_c=c, sections=[n, 128], fc_units=16)
           for n in (32, 64)}
    narrow = wl.make_weights(cfg[32])
    wide = np.zeros(wl.weight_count(cfg[64]), np.float32)
    small, large = wl.weight_slices(cfg[32]), wl.weight_slices(cfg[64])
    for name, (off, shape) in small.items():
        to, room = large[name]
        view = wide[to:to + int(np.prod(room))].reshape(room)
        view[tuple(slice(n) for n in shape)] = narrow[off:off + int(np.prod(shape))].reshape(shape)
    inputs = wl.make_batch(cfg[32], batch)
    print(f"case {frame} B={batch}", flush=True)
    want, _ = batch_bits.features(cfg[32], narrow, inputs)
    got, _ = batch_bits.features(cfg[64], wide, inputs)
    np.testing.assert_array_equal(got, want)
