"""Both ways that gen_features writes its planes, against the CPU oracle, bit
for bit.  By cells: boards of odd cell counts (or tensors that start inside 16
bytes) up to 350 cells and aligned ones whose planes leave lanes idle, up to
an output size; by planes: the same boards above that size, and the others.
Boards are taken around one, two and four 64-cell words, batches around the
changes of the waves per env (512 and 2,048 envs) and around the size limits.
Every value is an integer or is rounded once from double on both sides, so
the tolerance is zero."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


def bits(a):
    return np.ascontiguousarray(a).view(np.int32)


def make(H, W, P, E, seed, mode=None, **over):
    import paper_2606_23348_amd as gen
    mode = (0 if P == 2 else 2) if mode is None else mode
    prm = dict(mountain_thresh=workloads.mountain_thresh(1, 5), cities_min=min(2, H * W // 8),
               cities_max=min(6, H * W // 4), min_general_dist=min(4, (H + W) // 5), auto_reset=1)
    prm.update(over)
    b = gen.Batch(E, H, W, mode, gen.make_params(mode, P, **prm), seed=seed, with_obs=False)
    cfg = oracle.Config(H=H, W=W, mode=mode, P=P, seed=seed, env_base=0, **prm)
    return gen, b, cfg, oracle.reset(cfg, E)[0], oracle.feature_memory(E)


def compare(gen, b, cfg, ost, mem, steps, shift=0):
    import torch
    E, P, n = b.n_envs, b.P, b.n_envs * b.P * 38 * b.H * b.W
    raw = torch.full((n + 64,), 7.0, dtype=torch.float32, device="cuda")
    feat, tok = raw[shift:shift + n], torch.zeros((E, P, 2, 512), dtype=torch.float32, device="cuda")
    fmem = torch.zeros(gen.gen_feat_mem_bytes(b.st), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    b.sample(9, 0)
    for t in range(steps):
        gen.gen_features(b.st, fmem, feat, tok)
        want, wtok = oracle.features(cfg, ost, mem, tokens=True)
        assert np.array_equal(bits(feat.cpu().numpy().reshape(want.shape)), bits(want)), f"{b.H}x{b.W} P{P} E{E} step {t}"
        assert np.array_equal(tok.cpu().numpy(), wtok), f"tokens, step {t}"
        gen.gen_step_sample(b.st, b.actions, 9, t + 1, None, b.rewards, b.dones)
        oracle.step(cfg, ost, oracle.sample(cfg, ost, 9, t))
    edge = raw.cpu().numpy()
    assert (edge[:shift] == 7.0).all() and (edge[shift + n:] == 7.0).all()      # nothing written outside the tensor


@pytest.mark.parametrize("P", [2, 3, 5, 8])
@pytest.mark.parametrize("H,W,shift", [(3, 3, 0), (7, 9, 0), (8, 8, 0), (8, 8, 1), (5, 13, 2), (9, 15, 0), (11, 11, 0), (12, 20, 0),
                                       (13, 15, 3), (15, 17, 0), (16, 16, 1), (16, 16, 2), (13, 23, 0), (16, 20, 7), (17, 19, 0), (18, 19, 0), (13, 27, 1), (19, 21, 0)])
def test_small_batches(H, W, P, shift):
    compare(*make(H, W, P, 3, seed=H * W + P), steps=10, shift=shift)


@pytest.mark.parametrize("H,W,P,E", [(9, 9, 2, 512), (9, 9, 2, 513), (9, 9, 4, 2048), (9, 9, 4, 2049), (7, 9, 3, 2050), (8, 8, 3, 2060),
                                     (9, 9, 5, 2049), (13, 15, 7, 513), (15, 15, 8, 300), (17, 15, 2, 2049), (11, 13, 6, 260)])
def test_waves_per_env(H, W, P, E):
    compare(*make(H, W, P, E, seed=E), steps=3)


# bytes of the features: 152 E P H W; the limit of each kind of board between the two batches
@pytest.mark.parametrize("H,W,P,limit", [(9, 9, 3, 200), (11, 11, 8, 200), (11, 13, 2, 200), (13, 13, 4, 200), (13, 15, 3, 200),
                                         (13, 14, 7, 200), (8, 8, 3, 110), (10, 10, 3, 110), (10, 10, 4, 110), (10, 10, 4, 50), (13, 20, 5, 110), (17, 17, 2, 110),
                                         (13, 23, 6, 110), (17, 15, 8, 200)])
@pytest.mark.parametrize("above", [0, 1])
def test_at_the_size_limits(H, W, P, limit, above):
    E = limit * 1000000 // (152 * P * H * W) + above
    compare(*make(H, W, P, E, seed=E), steps=2)


@pytest.mark.parametrize("H,W,P,mode", [(9, 9, 2, 0), (13, 15, 4, 1), (24, 24, 2, 0)])
def test_sightings_older_than_the_age_table(H, W, P, mode):
    """Channel 21 beyond the table of 65,536 turns: the same episode 70,000 turns on."""
    import torch
    E = 4
    gen, b, cfg, ost, mem = make(H, W, P, E, seed=3, mode=mode, auto_reset=0)
    b.sample(9, 0)
    for t in range(120):
        b.features()
        want = oracle.features(cfg, ost, mem)
        gen.gen_step_sample(b.st, b.actions, 9, t + 1, None, b.rewards, b.dones)
        oracle.step(cfg, ost, oracle.sample(cfg, ost, 9, t))
    h = b.get_state()
    for jump in (65535, 4465):
        h["turn"] = h["turn"] + jump
        ost["turn"] += jump
        # nothing is visible to player 0: its sightings age
        for d in (h, ost):
            d["owner"][d["owner"] == 0] = -1
        b.set_state(h)
        b.features()
        want = oracle.features(cfg, ost, mem)
        torch.cuda.synchronize()
        assert np.array_equal(bits(b.feat.cpu().numpy()), bits(want)), f"jump {jump}"
    # log1p(120 + ...)/5 of a table entry is below 2.22; later ones are above
    assert (want[:, :, 21] > 2.22).any()


@pytest.mark.parametrize("fill", [0xA5, 0x7F, 0xFF])
@pytest.mark.parametrize("H,W,P,E,mode", [(23, 23, 2, 5, 0), (9, 15, 3, 4, 2), (16, 16, 4, 3, 1), (28, 32, 7, 2, 2), (10, 10, 2, 600, 0)])
def test_block_of_no_episode(H, W, P, E, mode, fill):
    """Memory that holds anything but this episode's header counts as empty."""
    import torch
    gen, b, cfg, ost, mem = make(H, W, P, E, seed=fill + P, mode=mode)
    feat = torch.zeros(E * P * 38 * H * W, dtype=torch.float32, device="cuda")
    fmem = torch.full((gen.gen_feat_mem_bytes(b.st),), fill, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    b.sample(9, 0)
    for t in range(10):
        gen.gen_features(b.st, fmem, feat)
        want = oracle.features(cfg, ost, mem)
        assert np.array_equal(bits(feat.cpu().numpy().reshape(want.shape)), bits(want)), f"step {t}"
        gen.gen_step_sample(b.st, b.actions, 9, t + 1, None, b.rewards, b.dones)
        oracle.step(cfg, ost, oracle.sample(cfg, ost, 9, t))
