"""gen_rollout over the batches and tensors that its callers have, against the
CPU oracle turn by turn: fewer waves an env (more than 256 envs), games
longer than the 512-turn scoreboard ring, and feature tensors that start
anywhere inside 16 bytes.  Every value is an integer or is rounded once from
double on both sides, so the tolerance is zero."""
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


def check(out, cfg, ost, mem, actor, t0, n, tokens):
    for t in range(n):
        want, wtok = oracle.features(cfg, ost, mem, tokens=True)
        assert np.array_equal(bits(out["feat"][t].cpu().numpy().reshape(want.shape)), bits(want)), f"features, turn {t0 + t}"
        if tokens:
            assert np.array_equal(out["tokens"][t].cpu().numpy(), wtok), f"tokens, turn {t0 + t}"
        act = oracle.sample(cfg, ost, actor, t0 + t)
        assert np.array_equal(out["actions"][t].cpu().numpy(), act), f"actions, turn {t0 + t}"
        r, d = oracle.step(cfg, ost, act)
        assert np.array_equal(out["rewards"][t].cpu().numpy(), r) and np.array_equal(out["dones"][t].cpu().numpy(), d)


@pytest.mark.parametrize("H,W,mode,P,E,T", [
    (10, 10, 0, 2, 260, 6), (23, 23, 0, 2, 300, 3), (24, 24, 0, 2, 512, 2), (12, 12, 2, 5, 260, 5), (13, 15, 2, 7, 300, 3),
    (9, 7, 2, 3, 700, 6), (12, 11, 2, 6, 258, 4), (25, 25, 2, 8, 258, 2), (32, 32, 1, 4, 257, 2), (13, 15, 1, 4, 1100, 2),
    (8, 8, 2, 3, 1100, 5), (16, 16, 0, 2, 2000, 2), (20, 12, 1, 4, 1200, 2), (31, 31, 0, 2, 520, 2)])
def test_many_envs(H, W, mode, P, E, T):
    import torch
    gen, b, cfg, ost, mem = make(H, W, mode, P, E, seed=E + P)
    for rep in range(2):
        out = b.rollout(T, 31, rep * T, tokens=True)
        torch.cuda.synchronize()
        check(out, cfg, ost, mem, 31, rep * T, T, True)
    st = b.get_state()
    for k in ost:
        assert np.array_equal(st[k], ost[k]), k


@pytest.mark.parametrize("E,mode,P", [(4, 0, 2), (259, 2, 3)])
def test_past_the_scoreboard_ring(E, mode, P):
    """Turns 512 and later of one launch reuse ring entries that other waves wrote earlier in the same launch."""
    import torch
    H, W, T = 8, 9, 545
    gen, b, cfg, ost, mem = make(H, W, mode, P, E, seed=5, auto_reset=0)
    n = E * P * 38 * H * W
    feat = torch.zeros((T, n), dtype=torch.float32, device="cuda")
    out = dict(feat=feat, tokens=torch.zeros((T, E, P, 2, 512), dtype=torch.float32, device="cuda"),
               actions=torch.zeros((T, E, P), dtype=torch.int32, device="cuda"),
               rewards=torch.zeros((T, E, P), dtype=torch.int32, device="cuda"),
               dones=torch.zeros((T, E), dtype=torch.uint8, device="cuda"))
    fmem = torch.zeros(gen.gen_feat_mem_bytes(b.st), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    gen.gen_rollout(b.st, fmem, T, 8, 0, out["feat"], out["actions"], out["rewards"], out["dones"], out["tokens"])
    torch.cuda.synchronize()
    for t in range(T):
        want, wtok = oracle.features(cfg, ost, mem, tokens=True)
        if t in (0, 1, 200, 400) or t >= 505:
            assert np.array_equal(out["tokens"][t].cpu().numpy(), wtok), f"tokens, turn {t}"
            assert np.array_equal(bits(feat[t].cpu().numpy().reshape(want.shape)), bits(want)), f"features, turn {t}"
        oracle.step(cfg, ost, oracle.sample(cfg, ost, 8, t))
    assert (ost["turn"] >= 540).any()


@pytest.mark.parametrize("shift", [1, 2, 3, 7])
@pytest.mark.parametrize("H,W,mode,P,E", [(11, 11, 0, 2, 5), (16, 16, 1, 4, 3), (17, 17, 2, 6, 3), (9, 15, 2, 3, 259), (23, 23, 0, 2, 2)])
def test_feature_tensor_off_16_bytes(H, W, mode, P, E, shift):
    """shift: floats between the tensor's start and a 256-byte boundary."""
    import torch
    T = 4
    gen, b, cfg, ost, mem = make(H, W, mode, P, E, seed=H + shift)
    n = T * E * P * 38 * H * W
    raw = torch.full((n + 16,), 7.0, dtype=torch.float32, device="cuda")
    out = dict(feat=raw[shift:shift + n].view(T, -1),
               actions=torch.zeros((T, E, P), dtype=torch.int32, device="cuda"),
               rewards=torch.zeros((T, E, P), dtype=torch.int32, device="cuda"),
               dones=torch.zeros((T, E), dtype=torch.uint8, device="cuda"))
    fmem = torch.zeros(gen.gen_feat_mem_bytes(b.st), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    gen.gen_rollout(b.st, fmem, T, 12, 0, out["feat"], out["actions"], out["rewards"], out["dones"])
    torch.cuda.synchronize()
    check(out, cfg, ost, mem, 12, 0, T, False)
    edge = raw.cpu().numpy()
    assert (edge[:shift] == 7.0).all() and (edge[shift + n:] == 7.0).all()


# bytes of a turn's features: 152 E P H W; the limit of each kind of board between the two batches
@pytest.mark.parametrize("H,W,mode,P,limit", [(15, 15, 2, 8, 110), (9, 9, 2, 5, 110), (11, 13, 1, 4, 110), (8, 8, 2, 3, 400), (17, 17, 1, 4, 60),
                                              (13, 23, 2, 6, 60)])
@pytest.mark.parametrize("above", [0, 1])
def test_at_the_size_limits(H, W, mode, P, limit, above):
    """Turns by cells up to the limit, by planes above it."""
    import torch
    E = limit * 1000000 // (152 * P * H * W) + above
    gen, b, cfg, ost, mem = make(H, W, mode, P, E, seed=E)
    out = b.rollout(2, 31, 0, tokens=True)
    torch.cuda.synchronize()
    check(out, cfg, ost, mem, 31, 0, 2, True)


@pytest.mark.parametrize("H,W,mode,P,E,T", [(23, 23, 0, 2, 3, 12), (15, 15, 2, 8, 3, 20), (16, 16, 2, 7, 3, 12), (17, 19, 1, 4, 300, 4), (15, 15, 2, 5, 400, 4),
                                            (9, 9, 1, 4, 513, 8), (8, 8, 0, 2, 600, 8), (3, 3, 0, 2, 40, 30), (5, 13, 2, 6, 270, 10)])
def test_boards_of_each_task(H, W, mode, P, E, T):
    import torch
    gen, b, cfg, ost, mem = make(H, W, mode, P, E, seed=T + P)
    for rep in range(2):
        out = b.rollout(T, 13, rep * T, tokens=True)
        torch.cuda.synchronize()
        check(out, cfg, ost, mem, 13, rep * T, T, True)


@pytest.mark.parametrize("H,W,mode,P,E", [(19, 21, 0, 2, 371), (19, 21, 0, 2, 372), (25, 25, 2, 8, 59), (25, 25, 2, 8, 60), (24, 24, 1, 4, 128),
                                          (24, 24, 1, 4, 129), (31, 31, 0, 2, 5), (19, 19, 2, 3, 7), (18, 31, 2, 5, 9), (23, 23, 2, 8, 260)])
def test_boards_of_three_rounds_and_more(H, W, mode, P, E):
    """On both sides of 45 MB of features a turn, and boards of 3 to 16 words."""
    import torch
    gen, b, cfg, ost, mem = make(H, W, mode, P, E, seed=E + P)
    for rep, tokens in enumerate((True, False)):
        out = b.rollout(4, 7, rep * 4, tokens=tokens)
        torch.cuda.synchronize()
        check(out, cfg, ost, mem, 7, rep * 4, 4, tokens)
