"""The staged observation writer, the cell bitmaps and the order-free moves at
the sizes where they change, against the CPU oracle, byte for byte: boards up
to 121 cells (a player a run) and beyond, 64, 128 and 192 quads of 4 cells and
a shifted one more, every remainder of the cell count by 4, tensors that start
inside a 128-byte line, 1 to 8 waves per env, and the batches and pools from
which aligned planes are staged."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
KEYS = ("owner", "army", "type", "turn", "episode", "alive", "finished", "gpos")


def params(H, W, P, **over):
    prm = dict(mountain_thresh=workloads.mountain_thresh(1, 5), cities_min=min(2, H * W // 8),
               cities_max=min(6, H * W // 4), min_general_dist=min(4, (H + W) // 5), auto_reset=1)
    prm.update(over)
    return prm


def check(H, W, mode, P, E, steps, off=0, padded=False, scoreboard=False, fused=True):
    import torch
    import paper_2606_23348_amd as gen
    prm, seed = params(H, W, P), 7 * H + W
    b = gen.Batch(E, H, W, mode, gen.make_params(mode, P, obs_layout=1 if padded else 0, **prm), seed=seed,
                  with_obs=False, scoreboard=scoreboard)
    cfg = oracle.Config(H=H, W=W, mode=mode, P=P, seed=seed, env_base=0, **prm)
    ost, _ = oracle.reset(cfg, E)
    PS = gen.plane_stride(H, W, P) if padded else H * W
    n = E * P * 8 * PS
    raw = torch.full((n + 256,), 77, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    obs = raw[off:off + n]

    def same(where):
        got = raw.cpu().numpy()
        assert (got[:off] == 77).all() and (got[off + n:] == 77).all(), where + ": written outside the tensor"
        planes = got[off:off + n].reshape(E, P, 8, PS)
        assert not planes[..., H * W:].any(), where + ": padding"
        assert np.array_equal(planes[..., :H * W].reshape(E, P, 8, H, W), oracle.observe(cfg, ost)), where

    gen.gen_observe(b.st, obs)
    same("observe")
    b.sample(3, 0)
    for t in range(steps):
        land = (b.land, b.army) if scoreboard else (None, None)
        if fused:
            gen.gen_step_sample(b.st, b.actions, 3, t + 1, obs, b.rewards, b.dones, *land)
        else:
            gen.gen_step(b.st, b.actions, obs, b.rewards, b.dones, *land)
            b.sample(3, t + 1)
        r, d = oracle.step(cfg, ost, oracle.sample(cfg, ost, 3, t))
        same(f"step {t}")
        assert np.array_equal(b.rewards.cpu().numpy(), r) and np.array_equal(b.dones.cpu().numpy(), d)
        if scoreboard:
            land, army = oracle.scoreboard(cfg, ost)
            assert np.array_equal(b.land.cpu().numpy(), land) and np.array_equal(b.army.cpu().numpy(), army)
    st = b.get_state()
    for k in KEYS:
        assert np.array_equal(st[k], ost[k]), k


BOARDS = [(3, 3, 2, 8), (3, 5, 0, 2), (5, 7, 1, 4), (11, 11, 2, 3), (9, 13, 0, 2), (6, 21, 1, 4), (11, 23, 0, 2), (5, 27, 2, 6),
          (15, 17, 0, 2), (21, 12, 0, 2), (17, 30, 1, 4), (19, 27, 2, 5), (22, 23, 0, 2), (25, 25, 2, 8), (29, 26, 0, 2), (31, 31, 2, 7),
          (30, 31, 1, 4)]


@pytest.mark.parametrize("off", [0, 16, 112])
@pytest.mark.parametrize("H,W,mode,P", BOARDS)
def test_odd_planes(H, W, mode, P, off):
    check(H, W, mode, P, 5, 6, off=off)


@pytest.mark.parametrize("E", [512, 513, 1025, 2049])
@pytest.mark.parametrize("H,W,mode,P", [(9, 7, 2, 7), (13, 10, 0, 2), (15, 9, 2, 5)])
def test_waves_by_batch(H, W, mode, P, E):
    check(H, W, mode, P, E, 2)


@pytest.mark.parametrize("H,W,mode,P,E,padded", [
    (18, 18, 0, 2, 5900, False), (17, 20, 1, 4, 2800, False), (32, 31, 0, 2, 1900, False), (16, 16, 1, 4, 3700, False),
    (19, 20, 0, 2, 4600, True), (21, 21, 1, 4, 28000, True)])
def test_aligned_planes_in_large_batches(H, W, mode, P, E, padded):
    """At least 30 MB of observation (400 MB for planes of 64-byte halves): staged; 16x16 never."""
    check(H, W, mode, P, E, 2, padded=padded)


@pytest.mark.parametrize("H,W,mode,P", [(11, 13, 2, 8), (9, 9, 1, 4), (16, 16, 2, 3)])
def test_scoreboard_and_separate_actor(H, W, mode, P):
    check(H, W, mode, P, 40, 12, scoreboard=True)
    check(H, W, mode, P, 40, 12, scoreboard=True, fused=False)


@pytest.mark.parametrize("H,W,P,E,padded", [(12, 12, 8, 8192, False), (12, 11, 5, 8191, False), (8, 16, 8, 8192, False),
                                            (11, 12, 5, 8192, False), (13, 13, 6, 16400, True)])
def test_more_than_four_players_in_large_batches(H, W, P, E, padded):
    """Aligned planes of more than 128 cells, 8,192 envs and more: fewer waves a CU."""
    check(H, W, 2, P, E, 1, padded=padded)


@pytest.mark.parametrize("off", [0, 16, 64])
@pytest.mark.parametrize("H,W,mode,P,E", [(24, 24, 0, 2, 4000), (16, 20, 2, 6, 2300), (28, 16, 1, 4, 2600), (32, 30, 2, 3, 2048), (32, 26, 0, 2, 2700)])
def test_planes_in_pairs(H, W, mode, P, E, off):
    """Planes that end in the middle of a line, two at a time (from 2,048 envs and 35 MB of observation on)."""
    assert E * P * 8 * H * W >= 35_000_000 and H * W % 128 == 64
    check(H, W, mode, P, E, 2, off=off)


def test_pool_from_64_megabytes():
    """A pool large enough for the staged writer (boards of 16x16 to 25x25, all
    modes): every env against the oracle, two steps."""
    import torch
    import paper_2606_23348_amd as gen
    n = 7000
    rng = np.random.default_rng(8)
    H, W = rng.integers(16, 26, n), rng.integers(16, 26, n)
    mode = rng.choice([0, 1, 2], n)
    P = np.where(mode == 0, 2, np.where(mode == 1, 4, rng.integers(2, 7, n)))
    specs = dict(H=H, W=W, mode=mode, P=P, cities_min=H * W // 72, cities_max=H * W // 48, min_general_dist=np.full(n, 4))
    pool = gen.Pool(specs, seed=12)
    assert pool.info.obs_bytes >= 64_000_000
    pool.reset(5)
    for _ in range(2):
        pool.step(5)
    torch.cuda.synchronize()
    obs = pool.obs.cpu().numpy()
    for e in rng.choice(n, 600, replace=False):
        h, w, p = int(H[e]), int(W[e]), int(P[e])
        prm = dict(mountain_thresh=gen.gen_default_params(0).mountain_thresh, cities_min=int(specs["cities_min"][e]),
                   cities_max=int(specs["cities_max"][e]), min_general_dist=4, auto_reset=1)
        cfg = oracle.Config(H=h, W=w, mode=int(mode[e]), P=p, seed=12, env_base=int(e), **prm)
        ost, _ = oracle.reset(cfg, 1)
        for t in range(2):
            oracle.step(cfg, ost, oracle.sample(cfg, ost, 5, t))
        got = gen.pool_env_obs(obs, int(pool.obs_off[e]), h, w, p)
        assert np.array_equal(got.reshape(1, p, 8, h, w), oracle.observe(cfg, ost)), f"env {e} {h}x{w} P {p}"
