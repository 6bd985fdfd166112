"""The single-launch decode runs every pass of a control step: the token of a
pass is chosen inside the launch and feeds the next pass.  Decoding freely and
decoding with the same tokens given must agree bit for bit (logits, tokens,
margins), for one, two and many passes per launch, and a second decode after
another prompt pass must repeat the first (nothing is left over in the
barrier counters, the accumulator or the weight ring)."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("cfg_fn", [synth.config_c1, synth.config_mid])
@pytest.mark.parametrize("n_decode", [2, 3, 12])
def test_free_and_given_tokens_agree(cfg_fn, n_decode):
    from paper_2608_10824_amd.session import Session
    cfg = cfg_fn().with_(n_decode=n_decode)
    s = Session(cfg, synth.model_weights(cfg, device=DEV), device=DEV)
    si = synth.step_inputs(cfg, cfg.n_patches // 2)
    fp, ids = si["frame_prev"].to(DEV), si["text_ids"].to(DEV)

    def decode(forced=None):
        s.step_prefill(fp, ids)
        t, m, lg = s.decode_actions(logits=True, forced_tokens=forced)
        torch.cuda.synchronize()
        return t.clone(), m.clone(), lg.clone()

    free = decode()
    given = decode(free[0])
    again = decode()
    for a, b, c in zip(free, given, again):
        assert torch.equal(a, b) and torch.equal(a, c)
    # each token is the highest action bin of the logits returned for it, and
    # another token in its place changes what follows
    lo = cfg.bin_lo
    assert torch.equal(free[0].long(), free[2][..., lo:].argmax(-1) + lo)
    other = free[0].clone()
    other[:, 0] = (other[:, 0] - lo + 1) % cfg.n_bins + lo
    moved = decode(other)
    assert torch.equal(moved[2][:, 0], free[2][:, 0]) and not torch.equal(moved[2][:, 1], free[2][:, 1])
    s.close()
