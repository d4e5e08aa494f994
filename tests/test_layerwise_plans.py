"""Host side of the layer-by-layer ResNet path: workspace and the choice of kernels."""
import itertools
import random

import pytest

from tests import host_program

MAIN = r"""
// the strip plans of a section: per plan LDS bytes of its largest map and of the launch, the most pixel tiles of a wavefront
// and the accumulators' limit, and whether the strips cover every row once
static void strips(const Section& sec)
{
    const int H = sec.PH, W = sec.PW, C = sec.conv0.Cout;
    strip_by_width(C, [&](auto cc) {
        using K = StripCfg<decltype(cc)::value>;
        auto tiles = [&](int r, int w) { return (K::tiles(r, w) + K::NPG - 1) / K::NPG; };
        StripBlockPlan b;
        if (b.choose<decltype(cc)::value>(H, W)) {
            int lds_rows = 0, most = 0;
            for (int s = 0; s < b.strips; ++s) {
                const int y0 = s * b.TH, ye = std::min(y0 + b.TH, H);
                const int ra = std::min(ye + 1, H) - std::max(y0 - 1, 0);
                lds_rows = std::max(lds_rows, ra + 2);
                most = std::max(most, tiles(ra, W));
            }
            const bool cover = (long)b.TH * b.strips >= H && (long)b.TH * (b.strips - 1) < H;
            const size_t asked = K::lds_bytes(b.conv_a_rows(b.TH, b.strips) + 2, W);
            printf("%zu %zu %d %d %d ", K::lds_bytes(lds_rows, W), asked, most, K::TPW, cover && asked <= RS_LDS_MAX);
        }
        const ConvLayer& c = sec.conv0;
        StripPoolPlan q;
        if (q.choose<decltype(cc)::value>(c.H, c.W, sec.PH, sec.pool_pad_h)) {
            int most = 0;
            for (int s = 0; s < q.strips; ++s) {
                const int p0 = s * q.PTH, p1 = std::min(p0 + q.PTH, sec.PH);
                const int n = std::min(2 * (p1 - 1) - sec.pool_pad_h + 3, c.H) - std::max(2 * p0 - sec.pool_pad_h, 0);
                most = std::max(most, n);
            }
            const bool cover = (long)q.PTH * q.strips >= sec.PH && (long)q.PTH * (q.strips - 1) < sec.PH && most <= q.rows;
            printf("%zu %zu %d %d %d", K::lds_bytes(q.rows + 2, c.W), RS_LDS_MAX, tiles(most, c.W), K::TPW, cover);
        }
        printf("\n");
        return true;
    });
}

int main()
{
    char what[8];
    int h, w, c, rows, n;
    while (scanf("%7s %d %d %d %d %d", what, &h, &w, &c, &rows, &n) == 6) {
        std::vector<int> sections(n);
        for (int& s : sections) if (scanf("%d", &s) != 1) return 1;
        const Plan p = resnet(h, w, c, sections);
        if (what[0] == 's') {
            strips(p.sections[0]);
        } else if (what[0] == 'b') {
            const LwLayout l = lw_layout(p, rows);
            printf("%zu %zu %zu %zu %zu\n", l.c0, l.u, l.r, l.x, l.end);
        } else {
            // a letter per section: strips, tiles, or neither; 256 compute units
            Bf16Packed o;
            bf16_pack(p, TORSO_NONE, (int)(p.flat + 31) / 32 * 32, 32, o);
            std::string route;
            for (int i = 0; i < n; ++i) {
                const LwSectionPlan pl = plan_lw_section(p.sections[i], &o.lw[5 * i], i == 0);
                route += strips_preferred(pl, sections[i], rows, 256) ? 'S' : pl.block.h ? 'T' : '-';
            }
            printf("%s\n", route.c_str());
        }
    }
}
"""

# frames (h, w, planes), sections, {rows: kernels of each section}: S strips, T tiles
ROUTES = [
    # the model-size variants
    ((72, 96, 3), (32, 64, 64), {1: "TTS", 64: "TTS", 256: "SSS", 4096: "SSS"}),
    ((72, 96, 3), (64, 128, 128), {1: "TSS", 32: "TSS", 64: "SSS", 1024: "SSS"}),
    ((90, 120, 16), (16, 32, 32, 32), {1: "TTSS", 256: "SSSS"}),
    ((108, 144, 16), (16, 32, 32, 32), {1: "TTSS", 256: "SSSS"}),
    # maps so wide that a strip is one or two rows: tiles, unless every strip has a compute unit of its own
    ((162, 216, 3), (64,), {1: "S", 16: "T", 256: "T"}),
    ((144, 192, 1), (64, 128), {2: "SS", 64: "ST", 256: "ST"}),
    ((160, 216, 3), (64, 128), {1: "SS", 64: "TT", 256: "TT"}),
    ((180, 400, 3), (32, 32), {1: "TT", 256: "TS"}),
    ((120, 800, 4), (16, 16), {1: "TT", 256: "TS"}),
    # strips of one section that end in a shorter one, two strips (one halo side each) and many
    ((116, 100, 3), (64,), {2: "T", 60: "S"}),
    ((124, 119, 1), (64, 128), {2: "TS", 60: "SS"}),
    ((139, 121, 4), (16, 16), {2: "TT", 200: "SS"}),
    # small whole images (5 x 3 pixels fill half of their pixel tiles)
    ((34, 22, 3), (32, 64, 128), {5: "SSS", 1541: "SSS"}),
    # one map, one strip, one tile; too wide for a strip
    ((40, 2, 4), (32, 64), {1: "SS", 500: "SS"}),
    ((18, 520, 1), (64, 128, 128), {2: "TTT", 300: "TTT"}),
    # no fused block at 48 channels
    ((50, 70, 3), (16, 48), {1: "T-", 300: "S-"}),
]


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
    out = program([f"buffers {h} {w} 3 {rows} {len(s)} {' '.join(map(str, s))}" for h, w, rows, s in cases])
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


def test_strips_are_chosen_where_they_are_faster(program):
    """Strips against tiles by the work of either plan and the workgroups a batch gives (both sides' times stand at
    strips_preferred)."""
    cases = [(*frame, rows, sections, route) for frame, sections, by_rows in ROUTES for rows, route in by_rows.items()]
    out = program([f"route {h} {w} {c} {rows} {len(s)} {' '.join(map(str, s))}" for h, w, c, rows, s, _ in cases])
    assert out == [c[-1] for c in cases], [(c, o) for c, o in zip(cases, out) if c[-1] != o]


def test_strips_fit_lds_and_the_accumulators(program):
    """A strip's map fits the LDS a workgroup asks for and its pixel tiles the accumulators (a wavefront with more would
    drop them), for every map and ragged strips, as the kernels work their rows out."""
    rng = random.Random(2)
    maps = [(1, 1), (2, 3), (9, 12), (17, 11), (36, 48), (54, 72), (2048, 2), (2, 500), (1, 1020), (300, 250)]
    maps += [(rng.randint(1, 200), rng.randint(1, 300)) for _ in range(300)]
    # (the pooling plan looks at conv0 as a layer of C input channels: planes do not matter)
    cases = [(2 * h - rng.randint(0, 1), 2 * w - rng.randint(0, 1), ch, rng.choice([1, 600, 1100, 1700, 2051, 5000]))
             for h, w in maps for ch in (16, 32, 64, 128)]
    out = program([f"strips {h} {w} 3 {rows} 1 {ch}" for h, w, ch, rows in cases])
    assert len(out) == len(cases)
    for case, line in zip(cases, out):
        v = list(map(int, line.split()))
        for lds, lds_max, tiles, tiles_max, cover in zip(*[iter(v)] * 5):
            assert lds <= lds_max and 1 <= tiles <= tiles_max and cover, (case, line)
    assert sum(len(line.split()) >= 5 for line in out) > len(out) // 2
