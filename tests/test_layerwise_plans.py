"""Host side of the layer-by-layer ResNet path: workspace."""
import itertools
import random

import pytest

from tests import host_program

MAIN = r"""
int main()
{
    int h, w, c, rows, n;
    while (scanf("%d %d %d %d %d", &h, &w, &c, &rows, &n) == 5) {
        std::vector<int> sections(n);
        for (int& s : sections) if (scanf("%d", &s) != 1) return 1;
        const LwLayout l = lw_layout(resnet(h, w, c, sections), rows);
        printf("%zu %zu %zu %zu %zu\n", l.c0, l.u, l.r, l.x, l.end);
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return host_program.build(tmp_path_factory.mktemp("plans"), MAIN)


def test_maps_that_live_together_do_not_overlap(program):
    """Every section's maps fit, and the second copy of the residual stream, which starts at the conv0 map, ends before
    R, which the block that reads it writes.  In frames of one row or column that copy is larger than the conv0 map (1 x
    5 frame, 16 channels: 160 bytes of map, 192 of x)."""
    rng = random.Random(1)
    frames = [(1, 1), (1, 2), (1, 5), (5, 1), (1, 1199), (2, 3), (3, 3), (7, 1), (1, 4095), (72, 96), (9, 9)]
    frames += [(rng.randint(1, 40), rng.randint(1, 40)) for _ in range(100)]
    cases = [(h, w, rng.choice([1, 3, 64, 2048]), s)
             for (h, w), s in itertools.product(frames, ([16], [16, 16], [16, 32, 64, 128], [64, 32, 16]))]
    out = program([f"{h} {w} 3 {rows} {len(s)} {' '.join(map(str, s))}" for h, w, rows, s in cases])
    assert len(out) == len(cases)
    up = lambda n: -(-n // 256) * 256  # noqa: E731
    for (h, w, rows, sections), line in zip(cases, out):
        c0, u, r, x, end = map(int, line.split())
        conv, pooled = [], []
        for ch in sections:
            ph, pw = (h + 1) // 2, (w + 1) // 2
            conv.append(rows * h * w * ch * 2)
            pooled.append(rows * ph * pw * ch * 2)
            h, w = ph, pw
        assert 2 * max(pooled) <= r
        assert c0 == 0 and u >= max(conv) and r - u >= max(pooled) and x - r >= max(pooled) and end - x >= 2 * max(pooled)
        assert end == up(max(conv)) + 2 * up(max(pooled)) + up(2 * max(pooled))     # no more memory than the maps
