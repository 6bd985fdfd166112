"""Stage 1 ranking where every static patch has its own cosine (sensor noise on
static patches), through the C ABI against the oracle, bit-exact: patch counts
around the 16 patches a workgroup ranks and the 64 it compares at a time, and
patches whose values take one load batch, several, and part of one."""
import numpy as np
import pytest
import torch

import synth
from oracle import patches as op

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("side,patch,views,batch", [(1, 14, 1, 1), (3, 5, 1, 2), (4, 14, 1, 1), (5, 16, 1, 3),
                                                    (9, 8, 2, 2), (17, 14, 1, 1), (31, 3, 1, 2), (32, 2, 1, 16)])
def test_ranks_of_noisy_static_patches(side, patch, views, batch):
    from paper_2608_10824_amd import gvc
    from paper_2608_10824_amd.session import desc_from
    L = 5
    cfg = synth.config_c1().with_(img=side * patch, patch=patch, n_views=views, batch=batch, n_layers=L,
                                  tau=(249, 250))
    rng = np.random.default_rng(side * 100 + patch)
    shape = (batch, views, cfg.img, cfg.img, 3)
    prev = rng.integers(0, 255, shape, dtype=np.uint8)
    cur = np.where(rng.random(shape) < 0.05, prev + 1, prev).astype(np.uint8)
    fresh = rng.integers(0, 255, shape, dtype=np.uint8)
    moved = rng.random((batch, views, side, 1, side, 1, 1)) < 0.3
    moved = np.broadcast_to(moved, (batch, views, side, patch, side, patch, 1)).reshape(batch, views, cfg.img, cfg.img, 1)
    cur = np.where(moved, fresh, cur)
    q = [1000, 800, 333, 17, 0]
    ft, fp = torch.from_numpy(cur).to(DEV), torch.from_numpy(prev).to(DEV)
    N = cfg.n_patches
    mask = torch.full((batch, L, N), 7, dtype=torch.uint8, device=DEV)
    n = torch.full((batch,), -1, dtype=torch.int32, device=DEV)
    gvc.select_static_noalloc(desc_from(cfg), ft.data_ptr(), fp.data_ptr(), 249, 250, q, mask.data_ptr(),
                              n.data_ptr(), torch.cuda.current_stream(DEV).cuda_stream)
    torch.cuda.synchronize()
    for b in range(batch):
        m, k, _, _ = op.select_static(cur[b], prev[b], patch, (249, 250), q)
        assert k == n[b].item()
        assert np.array_equal(mask[b].cpu().numpy().astype(bool), m)
