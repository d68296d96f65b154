"""Map generator at the edges of its row bitmaps and of its draw window,
against the CPU oracle, bit for bit: boards of 512 and 1,024 cells (the
window of draws behind the cells' starts empty), a few cells below (it holds
fewer draws than the generals need), rows of 32 cells, more cities than one
window of 64 draws holds, boards that run out of plain cells or of room, and
attempts that fail."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
KEYS = ("owner", "army", "type", "turn", "episode", "alive", "finished", "gpos")


@pytest.mark.parametrize("H,W,mode,P,over", [
    (16, 32, 0, 2, {}), (32, 32, 2, 8, {}), (32, 16, 1, 4, {}), (22, 23, 2, 7, {}), (17, 30, 1, 4, {}), (3, 32, 0, 2, {}),
    (32, 3, 0, 2, {}),
    (24, 24, 0, 2, dict(cities_min=70, cities_max=255)),
    (22, 23, 0, 2, dict(cities_min=40, cities_max=90)),
    (5, 6, 0, 2, dict(cities_min=28, cities_max=30, mountain_thresh=0)),
    (9, 9, 0, 2, dict(mountain_thresh=workloads.mountain_thresh(1, 2))),
    (6, 6, 0, 2, dict(mountain_thresh=2 ** 32 - 1)),
    (6, 7, 2, 8, dict(min_general_dist=6)),
    (8, 8, 0, 2, dict(min_general_dist=0)),
    (32, 32, 0, 2, dict(generator=1, min_general_dist=17, castle_radius=6, cities_min=9, cities_max=11)),
    (16, 32, 2, 8, dict(generator=1, min_general_dist=1, max_general_dist=7, castle_radius=2, cities_min=40, cities_max=60)),
    (12, 12, 0, 2, dict(generator=1, min_general_dist=0, max_general_dist=0, castle_radius=0, cities_min=1, cities_max=3)),
    (9, 8, 2, 4, dict(generator=1, min_general_dist=40, castle_radius=3)),
])
def test_mapgen_edges(H, W, mode, P, over):
    import torch
    import paper_2606_23348_amd as gen
    E, seed = 48, 1000 * H + W
    prm = dict(mountain_thresh=workloads.mountain_thresh(1, 5), cities_min=min(2, H * W // 8),
               cities_max=min(5, H * W // 4), min_general_dist=min(5, (H + W) // 4), auto_reset=1)
    prm.update(over)
    b = gen.Batch(E, H, W, mode, gen.make_params(mode, P, **prm), seed=seed, env_base=2 ** 33)
    want, _ = oracle.reset(oracle.Config(H=H, W=W, mode=mode, P=P, seed=seed, env_base=2 ** 33, **prm), E)
    torch.cuda.synchronize()
    got = b.get_state()
    for k in KEYS:
        assert np.array_equal(got[k], want[k]), f"{H}x{W} {over}: {k}"
