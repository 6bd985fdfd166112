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


@pytest.mark.parametrize("heads,head_dim", [(4, 64), (8, 64), (3, 128), (5, 128)])
def test_keys_and_values_of_another_decode_leave_no_trace(heads, head_dim):
    """Every pass appends a key and a value that the next passes of the same
    launch read back.  A decode of other tokens before this one leaves other
    keys and values at the same places: the results must equal those of a
    session that never ran it (heads on one compute die, or spread over
    several), bit for bit, and the per-step launches' within rounding."""
    import os
    from paper_2608_10824_amd.session import Session
    d = heads * head_dim if (heads * head_dim) % 256 == 0 else None
    cfg = synth.config_c1().with_(n_heads=heads, d_model=d or 256 * heads, n_decode=16)
    if not d:
        cfg = cfg.with_(n_heads=heads * 2)   # d a multiple of 256 keeps the single launch
    w = synth.model_weights(cfg, device=DEV)
    si = synth.step_inputs(cfg, cfg.n_patches // 2)
    fp, ids = si["frame_prev"].to(DEV), si["text_ids"].to(DEV)
    g = torch.Generator().manual_seed(heads)
    a, b = (torch.randint(0, cfg.vocab, (1, cfg.n_decode), generator=g, dtype=torch.int32).to(DEV) for _ in range(2))

    def decode(s, forced):
        s.step_prefill(fp, ids)
        t, m, lg = s.decode_actions(logits=True, forced_tokens=forced)
        torch.cuda.synchronize()
        return t.clone(), m.clone(), lg.clone()

    s1, s2 = Session(cfg, w, device=DEV), Session(cfg, w, device=DEV)
    os.environ["GVC_DECODE"] = "legacy"
    try:
        s3 = Session(cfg, w, device=DEV)
    finally:
        del os.environ["GVC_DECODE"]
    decode(s1, a)
    got, ref, step = decode(s1, b), decode(s2, b), decode(s3, b)
    for x, y in zip(got, ref):
        assert torch.equal(x, y)
    err = (got[2] - step[2]).norm(dim=-1) / step[2].norm(dim=-1)   # per position; bf16 roundings of two layers
    assert float(err.max()) <= 2e-2, err
    for s in (s1, s2, s3):
        s.close()


@pytest.mark.parametrize("layers,heads,head_dim,n_decode", [(1, 8, 64, 40), (1, 8, 64, 300), (1, 16, 128, 34),
                                                            (2, 8, 128, 140), (3, 24, 64, 90)])
def test_many_passes_of_a_launch_match_a_launch_per_pass(layers, heads, head_dim, n_decode):
    """Heads whose workgroups share a compute die exchange q, k and v through
    its caches.  A launch of many passes over few layers must read each pass's
    own: the keys and values appended must equal bit for bit those of launches
    of one pass each (GVC_DECODE_FLAGS=0, whose caches start empty), with short
    prompts, where nothing else pushes a line out, and with more layer steps
    than one launch takes (256); logits within the rounding of the two heads'
    sums."""
    from paper_2608_10824_amd import gvc
    from paper_2608_10824_amd.session import Session
    cfg = synth.config_c1().with_(n_layers=layers, n_heads=heads, d_model=heads * head_dim, img=28, n_text=4,
                                  n_decode=n_decode)
    w = synth.model_weights(cfg, device=DEV)
    si = synth.step_inputs(cfg, 2)
    fp, ids = si["frame_prev"].to(DEV), si["text_ids"].to(DEV)
    g = torch.Generator().manual_seed(layers * heads)
    fed = torch.randint(0, cfg.vocab, (1, n_decode), generator=g, dtype=torch.int32).to(DEV)

    def decode(flags, forced):
        with pytest.MonkeyPatch.context() as mp:
            if flags is not None:
                mp.setenv("GVC_DECODE_FLAGS", flags)
            s = Session(cfg, w, device=DEV)
        s.step_prefill(fp, ids)
        t, _, lg = s.decode_actions(logits=True, forced_tokens=forced)
        out = [t.clone(), lg.clone()] + [s.read(i, l).clone() for l in range(layers)
                                         for i in (gvc.STATE_K, gvc.STATE_V)]
        s.margin_gate()   # no barrier timed out
        s.close()
        return out

    got, ref = decode(None, fed), decode("0", fed)
    for x, y in zip(got[2:], ref[2:]):
        assert torch.equal(x, y)
    # The hidden states are the same, but the two final norms add the squares in
    # different orders (a few ulp), so about one value in 10^4 rounds to the
    # other bf16 neighbour: 2^-8 of a value.  Up to 4 such values of twice the
    # root mean square in a row of d move its logits by 2 * 2 * 2^-8 / sqrt(d).
    err = (got[1] - ref[1]).norm(dim=-1) / ref[1].norm(dim=-1)
    assert float(err.max()) <= 2 ** -6 / cfg.d_model ** 0.5, float(err.max())
    # freely chosen tokens of a decode that takes several launches feed back the same way
    free = decode(None, None)
    for x, y in zip(free, decode(None, free[0])):
        assert torch.equal(x, y)
