"""The tile GEMM at sizes where a tile can go wrong, through whole prompt
passes: row counts with a remainder in the last token block and tiles that are
partly or wholly padding, weight blocks and pairs that no shape divides (20, 65
and 60 blocks), an odd number of k steps, one token block.  A row's sum over k
does not depend on the tile, so every shape must give the same state bit for
bit: in one sum (every shape against the launcher's choice), and in slices
against split-k launches and the per-pair kernel."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
# (views, text, batch): prompt rows 73 (one episode, 16 of them recomputed), 201, 402 and 1005
SIZES = [(1, 9, 1), (3, 9, 1), (3, 9, 2), (3, 9, 5)]


def _states(cfg, w, si, envs):
    from paper_2608_10824_amd import gvc
    from paper_2608_10824_amd.session import Session
    fp, ft, ids = si["frame_prev"].to(DEV), si["frame_t"].to(DEV), si["text_ids"].to(DEV)
    out = []
    for env in envs:
        with pytest.MonkeyPatch.context() as mp:
            for k, v in env.items():
                mp.setenv(k, v)
            s = Session(cfg, w, device=DEV)
        s.step_prefill(fp, ids)
        s.decode_actions()
        s.margin_gate(force=[0] * cfg.batch)
        mask, _ = s.select_static(ft, fp)
        st = [s.read(gvc.STATE_H, cfg.n_layers).clone(), s.read(gvc.STATE_K, 1).clone()]
        s.step_prefill(ft, ids, None, mask)
        st += [s.read(i, l).clone() for i, l in ((gvc.STATE_H, 1), (gvc.STATE_H, cfg.n_layers), (gvc.STATE_K, 1),
                                                 (gvc.STATE_V, 1), (gvc.STATE_HEAD_LOGITS, 0))]
        out.append(st)
        s.close()
    return out


@pytest.mark.parametrize("views,text,batch", SIZES, ids=["73-rows", "201-rows", "402-rows", "1005-rows"])
def test_tile_shapes_agree_bit_for_bit(views, text, batch):
    cfg = synth.config_c1().with_(d_model=320, n_heads=5, ffn=1040, n_views=views, n_text=text, batch=batch,
                                  n_decode=2)
    w = synth.model_weights(cfg, device=DEV)
    si = synth.step_inputs(cfg, cfg.n_patches * 9 // 10)
    one = _states(cfg, w, si, [{"GVC_GEMM": "big"}] + [{"GVC_GEMM": "big", "GVC_BIG_TW": str(i)} for i in range(1, 11)])
    sliced = _states(cfg, w, si, [{"GVC_SK_TALL": "0"}, {}, {"GVC_SK_CORE": "0"}] +
                     [{"GVC_SK_CORE": "0", "GVC_BIG_TW": str(i)} for i in range(1, 6)])
    for name, runs in (("one sum", one), ("slices", sliced)):
        for i, r in enumerate(runs[1:], 1):
            for x, y in zip(r, runs[0]):
                assert torch.equal(x, y), (name, i)
    # the two orders of summation differ by fp32 rounding, which bf16 activations carry on
    for x, y in zip(one[0], sliced[0]):
        x, y = x.double(), y.double()
        assert float((x - y).norm() / y.norm()) <= 1e-2
