"""Rows of a large batch against the same rows alone: which kernels run depends on the batch, the bits do not."""
import numpy as np

import oracle
from paper_1910_06591_amd import seedinf, workloads as wl
from tests import host_program
from tests.parity import check_against_oracle, to_device

MAIN = r"""
// per line "rows h w planes sections...": the kernels of each section on 256 compute units, the first layer's (rows down the
// frame with their strips' height, or tile) before them.  Blocks: pair with images per workgroup or strips per image, strip, tile
int main()
{
    int B, h, w, c, n;
    while (scanf("%d %d %d %d %d", &B, &h, &w, &c, &n) == 5) {
        std::vector<int> sections(n);
        for (int& s : sections) if (scanf("%d", &s) != 1) return 1;
        const Plan p = resnet(h, w, c, sections);
        Bf16Packed o;
        bf16_pack(p, TORSO_NONE, (int)(p.flat + 31) / 32 * 32, 32, o);
        for (int i = 0; i < n; ++i) {
            const Section& sec = p.sections[i];
            const LwSectionPlan pl = plan_lw_section(sec, &o.lw[5 * i], i == 0);
            const bool strips = strips_preferred(pl, sections[i], B, 256);
            if (i == 0 && strips && first_rows_preferred(pl.first_rows, B, 256)) printf("rows%d ", pl.first_rows.h);
            else if (i == 0) printf("tile ");
            if (!strips) printf("tile ");
            else if (!pl.pair.TH) printf("strip ");
            else if (pl.pair.strips > 1) printf("pair:%d ", pl.pair.strips);
            else strip_by_width(sections[i], [&](auto cc) { printf("pair*%d ", pl.pair.stack<decltype(cc)::value>(B, sec.PH, sec.PW, 256)); return true; });
        }
        printf("\n");
    }
}
"""


def routes(tmp_path, cases):
    """The kernels of (rows, frame, sections), as MAIN names them."""
    out = host_program.build(tmp_path, MAIN)([f"{b} {h} {w} {c} {len(s)} {' '.join(map(str, s))}" for b, (h, w, c), s in cases])
    assert len(out) == len(cases)
    return [line.strip() for line in out]


def features(cfg, weights, inputs, rows=None):
    """Torso features of the step, and its outputs."""
    import torch
    batch = len(inputs["obs"])
    net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=batch), weights)
    out = net.step(**to_device(inputs))
    torch.cuda.synchronize()
    big = net.read_intermediate(0, batch).cpu().numpy()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    for row in rows or ():
        net.step(**to_device({k: None if v is None else np.ascontiguousarray(v[[row]]) for k, v in inputs.items()}))
        np.testing.assert_array_equal(net.read_intermediate(0, 1).cpu().numpy()[0], big[row], err_msg=f"row {row}")
    net.close()
    return big, got


def check(orc, frame, sections, batch):
    """Torso features of the large batch equal those of its rows in batches of one, and its outputs the oracle: every place
    of the first stack of images and of the last."""
    h, w, c = frame
    cfg = dict(wl.CONFIGS["C3"], label=f"{h}x{w}x{c}, sections {sections}", index=131, obs_h=h, obs_w=w, obs_c=c, sections=list(sections), fc_units=16)
    weights, inputs = wl.make_weights(cfg), wl.make_batch(cfg, batch)
    print(f"case {cfg['label']} B={batch}", flush=True)
    rows = [0, 1, 2, 3, batch // 2, *range(batch - 4, batch)]
    _, got = features(cfg, weights, inputs, rows)
    pick = lambda v: None if v is None else np.ascontiguousarray(v[rows])  # noqa: E731
    ref = orc.forward(oracle.make_arch(cfg), weights, pick(inputs["obs"]), **{k: pick(inputs[k]) for k in ("prev_action", "prev_reward", "h_in", "c_in", "uniforms")})
    check_against_oracle({k: v[rows] for k, v in got.items()}, ref, 2e-2, pick(inputs["uniforms"]))
