"""The feature planes and the rollout kernel at the sizes where their layout
changes, against the CPU oracle, bit for bit: boards around 121 cells (two
players share a wave below), around 64, 128 and 192 quads of 4 cells (rounds
of a plane), of 1,024 cells and 8 players (the most LDS), with planes on and
off 16- and 128-byte boundaries (odd cell counts, a tensor that starts inside
one), odd player counts, and batches of one env.  Every value is an integer
or is rounded once from double on both sides, so the tolerance is zero."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


def bits(a):
    return np.ascontiguousarray(a).view(np.int32)


def make(H, W, mode, P, E, seed, **over):
    import paper_2606_23348_amd as gen
    prm = dict(mountain_thresh=workloads.mountain_thresh(1, 5), cities_min=min(2, H * W // 8),
               cities_max=min(6, H * W // 4), min_general_dist=min(4, (H + W) // 5), auto_reset=1)
    prm.update(over)
    b = gen.Batch(E, H, W, mode, gen.make_params(mode, P, **prm), seed=seed)
    cfg = oracle.Config(H=H, W=W, mode=mode, P=P, seed=seed, env_base=0, **prm)
    return gen, b, cfg, oracle.reset(cfg, E)[0], oracle.feature_memory(E)


BOARDS = [(3, 3, 2, 8), (5, 5, 2, 3), (11, 11, 2, 3), (11, 11, 0, 2), (10, 12, 1, 4), (4, 31, 2, 5), (12, 12, 2, 7), (8, 31, 0, 2),
          (15, 17, 1, 4), (16, 16, 0, 2), (17, 17, 0, 2), (16, 31, 0, 2), (22, 22, 1, 4), (16, 32, 0, 2), (23, 23, 2, 5),
          (24, 31, 0, 2), (25, 30, 2, 3), (24, 32, 0, 2), (27, 29, 0, 2), (32, 32, 2, 8), (31, 31, 1, 4)]


@pytest.mark.parametrize("H,W,mode,P", BOARDS)
@pytest.mark.parametrize("shift", [0, 1, 2, 7])
def test_planes(H, W, mode, P, shift):
    """shift: floats between the tensor's start and a 256-byte boundary."""
    import torch
    E = 3
    gen, b, cfg, ost, mem = make(H, W, mode, P, E, seed=H + 40 * W)
    n = E * P * 38 * H * W
    raw = torch.full((n + 16,), 7.0, dtype=torch.float32, device="cuda")
    feat = raw[shift:shift + n]
    fmem = torch.zeros(gen.gen_feat_mem_bytes(b.st), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    b.sample(9, 0)
    for t in range(11):
        gen.gen_features(b.st, fmem, feat)
        want = oracle.features(cfg, ost, mem)
        assert np.array_equal(bits(feat.cpu().numpy().reshape(want.shape)), bits(want)), f"{H}x{W} P{P} step {t}"
        b.step_sample(9, t + 1)
        oracle.step(cfg, ost, oracle.sample(cfg, ost, 9, t))
    edge = raw.cpu().numpy()
    assert (edge[:shift] == 7.0).all() and (edge[shift + n:] == 7.0).all()      # nothing written outside the tensor


@pytest.mark.parametrize("H,W,mode,P,E", [(10, 10, 0, 2, 1100), (16, 16, 1, 4, 1030), (9, 7, 2, 8, 1040), (24, 24, 0, 2, 1030),
                                             (12, 11, 2, 3, 256), (12, 11, 2, 3, 257), (25, 25, 2, 8, 258),
                                             (31, 31, 1, 4, 258), (32, 31, 0, 2, 260), (32, 32, 2, 8, 257)])
def test_waves_per_env(H, W, mode, P, E):
    """More than 1,024 envs: 2, 4 or 8 waves per env by the board's LDS; 16 up to 256 envs."""
    gen, b, cfg, ost, mem = make(H, W, mode, P, E, seed=E)
    b.sample(9, 0)
    for t in range(4):
        b.features(tokens=True)
        want, wtok = oracle.features(cfg, ost, mem, tokens=True)
        assert np.array_equal(bits(b.feat.cpu().numpy()), bits(want)) and np.array_equal(b.tokens.cpu().numpy(), wtok)
        b.step_sample(9, t + 1)
        oracle.step(cfg, ost, oracle.sample(cfg, ost, 9, t))


@pytest.mark.parametrize("H,W,mode,P,E,T,over", [
    (23, 23, 0, 2, 5, 12, dict(generator=1, min_general_dist=17, castle_radius=6, cities_min=9, cities_max=11)),
    (32, 32, 2, 8, 2, 10, {}),
    (11, 11, 2, 3, 1, 20, {}),
    (17, 12, 1, 4, 6, 30, {}),
    (4, 4, 2, 3, 24, 120, dict(cities_min=0, cities_max=1, min_general_dist=2)),             # many episodes
    (4, 4, 2, 3, 24, 90, dict(cities_min=0, cities_max=1, min_general_dist=2, auto_reset=0)),  # frozen games
    (16, 32, 0, 2, 3, 9, {}),
])
def test_rollout_in_one_launch(H, W, mode, P, E, T, over):
    """Rollouts before and after plain features calls on the same memory."""
    import torch
    gen, b, cfg, ost, mem = make(H, W, mode, P, E, seed=3 * H + W, **over)
    actor, t0 = 55, 0
    for rep, n in enumerate((3, T, 1)):
        out = b.rollout(n, actor, t0, tokens=rep != 2)
        torch.cuda.synchronize()
        for t in range(n):
            want, wtok = oracle.features(cfg, ost, mem, tokens=True)
            assert np.array_equal(bits(out["feat"][t].cpu().numpy()), bits(want)), f"rollout {rep} t {t}"
            if rep != 2:
                assert np.array_equal(out["tokens"][t].cpu().numpy(), wtok), f"rollout {rep} tokens {t}"
            act = oracle.sample(cfg, ost, actor, t0 + t)
            assert np.array_equal(out["actions"][t].cpu().numpy(), act), f"rollout {rep} actions {t}"
            r, d = oracle.step(cfg, ost, act)
            assert np.array_equal(out["rewards"][t].cpu().numpy(), r) and np.array_equal(out["dones"][t].cpu().numpy(), d)
        t0 += n
        st = b.get_state()
        for k in ost:
            assert np.array_equal(st[k], ost[k]), f"rollout {rep}: {k}"
        feat = torch.zeros((E, P, 38, H, W), dtype=torch.float32, device="cuda")
        tok = torch.zeros((E, P, 2, 512), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        gen.gen_features(b.st, b.fmem, feat, tok)      # Batch.features() would start a memory of its own here
        want, wtok = oracle.features(cfg, ost, mem, tokens=True)
        assert np.array_equal(bits(feat.cpu().numpy()), bits(want)) and np.array_equal(tok.cpu().numpy(), wtok)


@pytest.mark.parametrize("P", [2, 3, 5, 8])
@pytest.mark.parametrize("H,W", [(16, 16), (12, 19), (15, 15), (17, 17), (15, 30), (22, 22), (9, 25), (23, 21)])
def test_two_players_to_a_task(H, W, P):
    """One and two rounds of 64 quads (and the boards next to them), odd player counts: the last task has one player."""
    import torch
    E = 2
    gen, b, cfg, ost, mem = make(H, W, 2, P, E, seed=H * W + P)
    fmem = torch.zeros(gen.gen_feat_mem_bytes(b.st), dtype=torch.uint8, device="cuda")
    n = E * P * 38 * H * W
    raw = torch.full((n + 64,), 7.0, dtype=torch.float32, device="cuda")
    feat = raw[3:3 + n] if W % 3 == 0 else raw[:n]
    torch.cuda.synchronize()
    b.sample(9, 0)
    for t in range(9):
        gen.gen_features(b.st, fmem, feat)
        want = oracle.features(cfg, ost, mem)
        assert np.array_equal(bits(feat.cpu().numpy().reshape(want.shape)), bits(want)), f"step {t}"
        b.step_sample(9, t + 1)
        oracle.step(cfg, ost, oracle.sample(cfg, ost, 9, t))
    got = raw.cpu().numpy()
    lo = 3 if W % 3 == 0 else 0
    assert (got[:lo] == 7.0).all() and (got[lo + n:] == 7.0).all()
