"""The head's token and margin where a row of logits is cut into parts (more
than 4096 logits) and where it is not: greedy bin token equal to the returned
logits' argmax (ties to the lower id), margin against a float64 softmax of
them, over the whole vocabulary and over the bins, decoding in parallel, one
episode by one launch and three by per-step launches; twice, so that the parts'
tickets are left as they were found."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("vocab", [1024, 4096, 4112, 12304, 32000])
@pytest.mark.parametrize("mode", ["chunk", "single", "batch"])
@pytest.mark.parametrize("full", [True, False])
def test_tokens_and_margins_of_the_returned_logits(vocab, mode, full):
    from paper_2608_10824_amd.session import Session
    cfg = synth.config_c4_tiny() if mode == "chunk" else synth.config_c1().with_(n_decode=3,
                                                                                 batch=3 if mode == "batch" else 1)
    cfg = cfg.with_(vocab=vocab, norm_full_vocab=full, bin_scale_log2=-2)
    s = Session(cfg, synth.model_weights(cfg, device=DEV), device=DEV)
    si = synth.step_inputs(cfg, 20)
    fp, ids = si["frame_prev"].to(DEV), si["text_ids"].to(DEV)
    ex = si["extra_rows"].to(DEV) if si["extra_rows"] is not None else None
    for _ in range(2):
        s.step_prefill(fp, ids, ex)
        tok, mg, lg = s.decode_actions(logits=True)
        torch.cuda.synchronize()
        lg64 = lg.double()
        lo = cfg.bin_lo
        assert torch.equal(tok.long(), lg64[..., lo:].argmax(-1) + lo)
        p = torch.softmax(lg64 if full else lg64[..., lo:], dim=-1)[..., (lo if full else 0):]
        top = p.topk(2, dim=-1).values
        # fp32 exp and sums of up to 32000 terms: a few ulp of each probability
        assert float(((top[..., 0] - top[..., 1]) - mg.double()).abs().max()) <= 4e-6
    s.close()


@pytest.mark.parametrize("vocab", [1024, 12304, 32000])
@pytest.mark.parametrize("mode", ["chunk", "single", "batch"])
@pytest.mark.parametrize("first,n", [(66, 1), (64, 4), (64, 16), (0, 512)])
def test_not_a_number_among_the_logits_reaches_the_margins(vocab, mode, first, n):
    """Logits that are not numbers, outside the bins, as one value, as all that a
    thread of the reduction sees and as all of whole waves: the softmax has no
    value, so every margin is NaN and the gate fires; over the bins alone they
    do not count."""
    from paper_2608_10824_amd.session import Session
    cfg = synth.config_c4_tiny() if mode == "chunk" else synth.config_c1().with_(n_decode=3,
                                                                                 batch=3 if mode == "batch" else 1)
    for full in (True, False):
        cfg = cfg.with_(vocab=vocab, norm_full_vocab=full)
        w = synth.model_weights(cfg, device=DEV)
        w["lm_head"][first:first + n] = float("nan")
        s = Session(cfg, w, device=DEV)
        si = synth.step_inputs(cfg, 20)
        s.step_prefill(si["frame_prev"].to(DEV), si["text_ids"].to(DEV),
                       si["extra_rows"].to(DEV) if si["extra_rows"] is not None else None)
        _, mg, lg = s.decode_actions(logits=True)
        torch.cuda.synchronize()
        assert bool(lg[..., first:first + n].isnan().all()) and int(lg.isnan().sum()) == n * cfg.batch * cfg.n_decode
        assert bool((mg.isnan() if full else mg.isfinite()).all()), mg
        if full:
            assert all(s.margin_gate()[1])
        s.close()
