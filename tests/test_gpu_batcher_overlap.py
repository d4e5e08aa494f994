"""The batcher's overlapped transfers: frames sent while rows are added and torsos started chunk by chunk give the step's bits."""
import numpy as np
import pytest

from paper_1910_06591_amd import seedinf, workloads as wl

pytestmark = pytest.mark.gpu


NETS = {
    "C2": dict(wl.CONFIGS["C2"], index=61),               # greedy, with epsilon-greedy exploration
    "C3": dict(wl.CONFIGS["C3"], index=61),
    "C4": dict(wl.CONFIGS["C4"], index=61),
    # layer by layer; 13 x 15 x 16 features: rows padded to whole chunks of 32
    "layers": dict(wl.CONFIGS["C3"], label="50x60x3, sections 16 16", obs_h=50, obs_w=60, sections=[16, 16], index=61),
}


@pytest.mark.parametrize("depth", [1, 2])
@pytest.mark.parametrize("name", ["C2", "C3", "C4", "layers"])
def test_rounds_equal_steps(name, depth):
    """Rounds of whole chunks, ragged ones, rows added one by one and in groups, and reserved rows written only before the
    submit (which hold the frames back): actions and states are those of seed_infer_step on the same rows.  One round
    at a time the frames travel while rows are added and the torso starts chunk by chunk (700 rows: 512, then
    188); with a batch in flight they go at the submit."""
    import torch
    cfg = NETS[name]
    n, A, Hn = 700, cfg["num_actions"], cfg["lstm_units"]
    rng = np.random.default_rng(5)
    weights = wl.make_weights(cfg, bf16_representable=True)
    net = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=n), weights)
    ref = seedinf.SeedInfer(seedinf.make_arch(cfg, max_batch=n), weights)
    bat = seedinf.Batcher(net, n)
    frames = wl.make_obs(cfg, n, seed=7)
    h, c = (torch.zeros(n, max(Hn, 1), device="cuda") for _ in range(2))
    last = torch.zeros(n, dtype=torch.int32, device="cuda")

    def check(item):
        ticket, actors, args = item
        idx = torch.from_numpy(actors).long().cuda()
        got = bat.wait(ticket)
        rec = dict(prev_action=last[idx], prev_reward=args["rewards"], h_in=h[idx], c_in=c[idx], done=args["dones"]) if Hn else {}
        out = ref.step(args["obs"], **args["select"], **rec)
        np.testing.assert_array_equal(got, out["action"].cpu().numpy())
        last[idx] = out["action"]
        if Hn:
            h[idx], c[idx] = out["h"], out["c"]

    pending = []
    for rows, plan in ((700, "many"), (512, "many"), (256, "groups"), (300, "reserve"), (257, "one"), (3, "many"), (700, "groups")):
        actors = rng.permutation(n)[:rows].astype(np.int32)
        pick = rng.integers(0, n, rows)
        obs, rew, dn = frames[pick], rng.standard_normal(rows).astype(np.float32), (rng.random(rows) < 0.1).astype(np.uint8)
        if cfg["select"] == 1:
            select = dict(uniforms=wl.make_uniforms(cfg, rows, seed=int(rng.integers(1 << 30))))
        else:
            select = dict(epsilon=rng.random(rows, dtype=np.float32) * np.float32(0.5), explore_uniforms=rng.random((rows, 2), dtype=np.float32))
        print(f"{name} rows {rows} {plan}", flush=True)
        if plan == "one":
            for i in range(rows):
                bat.add(int(actors[i]), obs[i], float(rew[i]), bool(dn[i]))
        else:
            cut = {"many": [0, rows], "groups": [0, 1, rows // 3, rows], "reserve": [0, 150, rows]}[plan]
            slots = []
            for i0, i1 in zip(cut, cut[1:]):
                if plan == "reserve" and i0:
                    slots.append((bat.reserve(int(actors[i0]), float(rew[i0]), bool(dn[i0])), i0))
                    i0 += 1
                bat.add_many(actors[i0:i1], obs[i0:i1], rew[i0:i1], dn[i0:i1])
            for slot, i in slots:
                slot[...] = obs[i]
        args = dict(obs=torch.from_numpy(obs).cuda(), rewards=torch.from_numpy(rew).cuda(), dones=torch.from_numpy(dn).cuda(),
                    select={k: torch.from_numpy(v).cuda() for k, v in select.items()})
        pending.append((bat.submit(**select), actors, args))
        if len(pending) == depth:
            check(pending.pop(0))
    while pending:
        check(pending.pop(0))
    if Hn:
        for a in (0, n // 2, n - 1):
            hh, cc = bat.read_state(a)
            np.testing.assert_array_equal(hh, h[a].cpu().numpy())
            np.testing.assert_array_equal(cc, c[a].cpu().numpy())
    for x in (bat, net, ref):
        x.close()
