"""Owner bytes that are no player.  gen_set_state refuses them, but a caller's
own writes to the documented device layout may hold them: the totals and the
feature masks, which are addressed by the owner, leave them out, and the cells
around them keep their values.  Expected values from the definitions in numpy."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
ODD = (8, 9, 33, 40, 64, 100, 127)


@pytest.mark.parametrize("H,W,mode,P", [(16, 16, 0, 2), (25, 25, 2, 8), (9, 11, 1, 4), (32, 32, 2, 8)])
def test_owner_bytes_that_are_no_player(H, W, mode, P):
    import torch
    import paper_2606_23348_amd as gen
    E, HW = 4, H * W
    prm = dict(mountain_thresh=workloads.mountain_thresh(1, 5), cities_min=2, cities_max=4, min_general_dist=3, auto_reset=1)
    b = gen.Batch(E, H, W, mode, gen.make_params(mode, P, **prm), seed=6, scoreboard=True)
    cfg = oracle.Config(H=H, W=W, mode=mode, P=P, seed=6, env_base=0, **prm)
    ost = oracle.reset(cfg, E)[0]
    for t in range(30):
        b.sample(3, t)
        b.step()
        oracle.step(cfg, ost, oracle.sample(cfg, ost, 3, t))
    st = b.st
    owner = b.buf[st.off_owner:st.off_owner + E * st.stride].view(torch.int8).view(E, st.stride)
    army = b.buf[st.off_army:st.off_army + 4 * E * st.stride].view(torch.int32).view(E, st.stride)
    own, arm = ost["owner"].reshape(E, HW).copy(), ost["army"].reshape(E, HW).copy()
    free = np.argwhere((own[0] < 0) & (ost["type"].reshape(E, HW)[0] == 0))[:len(ODD), 0]
    own[0, free], arm[0, free] = ODD[:len(free)], 1000 + np.arange(len(free))
    owner[:, :HW] = torch.as_tensor(own).cuda()
    army[:, :HW] = torch.as_tensor(arm).cuda()
    torch.cuda.synchronize()
    land = np.stack([(own == p).sum(1) for p in range(P)], 1)
    tot = np.stack([np.where(own == p, arm, 0).astype(np.int64).sum(1) for p in range(P)], 1)

    b.features(tokens=True)
    f = b.feat.cpu().numpy().reshape(E, P, 38, HW)
    for p in range(P):
        mine = own == p
        assert np.array_equal(f[:, p, 10] > 0, mine) and np.array_equal(f[:, p, 1], np.where(mine, arm, 0))
        assert np.array_equal(f[:, p, 24], np.where(mine, arm, 0))             # no earlier frame
        foe = (own >= 0) & ~mine & ~((mode == 1) & (own == (p ^ 2))) & (f[:, p, 12] == 0)
        assert np.array_equal(f[:, p, 11] > 0, foe) and np.array_equal(f[:, p, 2], np.where(foe, arm, 0))
        assert np.array_equal(f[:, p, 16, 0], land[:, p]) and np.array_equal(f[:, p, 17, 0], tot[:, p])
        them = [q for q in range(P) if q != p and not (mode == 1 and q == (p ^ 2))]
        assert np.array_equal(f[:, p, 18, 0], land[:, them].sum(1)) and np.array_equal(f[:, p, 19, 0], tot[:, them].sum(1))

    b.actions.zero_()
    torch.cuda.synchronize()
    b.step()                                                                   # turn 31: nothing grows, nobody moves
    torch.cuda.synchronize()
    assert np.array_equal(b.land.cpu().numpy(), land) and np.array_equal(b.army.cpu().numpy(), tot)
    assert np.array_equal(owner[:, :HW].cpu().numpy(), own) and np.array_equal(army[:, :HW].cpu().numpy(), arm)

    out = b.rollout(1, 5, 31)
    torch.cuda.synchronize()
    f = out["feat"][0].cpu().numpy().reshape(E, P, 38, HW)
    for p in range(P):
        assert np.array_equal(f[:, p, 10] > 0, own == p)
        assert np.array_equal(f[:, p, 16, 0], land[:, p]) and np.array_equal(f[:, p, 17, 0], tot[:, p])
