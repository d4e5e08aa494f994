"""The first layer pooled down its rows: strips on the CPU, the kernel against the tile kernel and the oracle."""
import random

import pytest

from tests import batch_bits, host_program

MAIN = r"""
// per frame: LDS bytes, items of a strip's input and registers for them, and whether the strips cover the pooled rows once
int main()
{
    int H, W, cin, cout;
    while (scanf("%d %d %d %d", &H, &W, &cin, &cout) == 4) {
        ConvLayer c{};
        c.Cin = cin; c.Cout = cout;
        LwLayerDev d{};
        d.first_off = 0;
        const bool any = first_rows_by_layer(d, c, [&](auto ci, auto co) {
            using K = FirstRowsCfg<decltype(ci)::value, decltype(co)::value>;
            int h = 0, n = 0;
            const int PH = (H + 1) / 2;
            if (!K::choose(PH, W, h, n)) return false;
            printf("%zu %d %d %d\n", K::lds_bytes(h, W), K::items(2 * h + 3, W), K::PRE * FR_THREADS, (long)h * n >= PH && (long)h * (n - 1) < PH);
            return true;
        });
        if (!any) printf("-\n");
    }
}
"""


def test_strips_fit_lds_and_the_registers(tmp_path):
    rng = random.Random(4)
    frames = [(1, 1), (1, 4), (72, 96), (108, 144), (90, 120), (2, 4096), (400, 8)]
    frames += [(rng.randint(1, 200), rng.randint(1, 120) * rng.choice([1, 4])) for _ in range(200)]
    cases = [(h, w, ci, co) for h, w in frames for ci in (1, 3, 4, 16) for co in (16, 32, 64)]
    out = host_program.build(tmp_path, MAIN)([" ".join(map(str, c)) for c in cases])
    assert len(out) == len(cases)
    for case, line in zip(cases, out):
        if line != "-":
            lds, items, most, cover = map(int, line.split())
            assert lds <= 80 * 1024 and items <= most and cover and (case[2] == 16 or case[1] % 4 == 0), (case, line)
    assert sum(line != "-" for line in out) > len(out) // 3


# frames, section, rows; the kernels at that many rows and at one (first layer, blocks)
CASES = [
    ((72, 96, 3), (32,), 131, "rows9 pair:2", "tile tile"),                # four strips
    ((73, 100, 4), (64,), 60, "rows4 strip", "tile tile"),                 # odd height: a padded row above; a last column strip of four pixels
    ((31, 44, 1), (16,), 600, "rows16 pair*3", "tile pair*1"),             # one strip, 22 pooled columns
    ((57, 61, 16), (16,), 300, "rows10 pair*2", "tile tile"),              # odd both ways, 16 planes
    ((50, 34, 16), (32,), 300, "rows13 pair*2", "tile pair*1"),
    ((50, 60, 1), (32,), 300, "rows13 pair*1", "tile tile"),
    ((60, 64, 4), (16,), 300, "rows15 pair*2", "tile tile"),
    ((36, 60, 16), (64,), 300, "rows5 pair*1", "tile tile"),
    ((20, 200, 3), (64,), 131, "rows2 strip", "tile strip"),               # the thinnest strips: two pooled rows
    ((20, 240, 16), (16,), 300, "rows2 pair*1", "tile tile"),
    ((2, 4, 3), (16,), 512, "tile pair*2", "tile pair*1"),                 # one pooled row: stays on the tile kernel
    ((40, 400, 3), (32,), 64, "tile tile", "tile tile"),                   # blocks on tiles: so does the first layer
]


def test_cases_take_the_kernels_they_compare(tmp_path):
    out = batch_bits.routes(tmp_path, [(b, f, s) for f, s, rows, *_ in CASES for b in (rows, 1)])
    assert list(zip(out[::2], out[1::2])) == [(many, one) for *_, many, one in CASES]


@pytest.mark.gpu
@pytest.mark.parametrize("frame,sections,batch", [c[:3] for c in CASES], ids=str)
def test_pooling_down_the_rows_gives_the_tile_kernels_bits(orc, frame, sections, batch):
    batch_bits.check(orc, frame, sections, batch)
