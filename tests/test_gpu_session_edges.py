"""A session's forwards where their bookkeeping ends."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rt():
    from paper_2512_21857_amd import runtime
    assert torch.cuda.is_available()
    return runtime


def _session(rt, dtype, **kw):
    cfg = synth.shrink(synth.get_config("tiny"), dtype=dtype)
    return cfg, rt.DeviceSession(rt.DeviceModel(cfg, synth.model_weights(cfg)), cfg, **kw)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("call,short", [("verify", "resid_elems"), ("verify", "meta_elems"), ("expand", "resid_elems"),
                                        ("expand", "xin_bytes"), ("expand", "meta_elems")])
def test_full_capture_buffer_launches_nothing(rt, dtype, call, short):
    """A forward whose record would overrun a capture buffer fails with the capacity code and
    leaves every byte of the session's workspace, caches and record as it was."""
    from paper_2512_21857_amd import abi
    cfg, sess = _session(rt, dtype)
    sess.prefill(synth.prefix_ids(cfg))
    sess.expand(2, 3, 9)
    sess.verify()
    if call == "verify":
        sess.expand(1, 4, 16)   # other rows than the last verify's, so that a launch shows
    sess.set_capture(**{**dict(resid_elems=1 << 20, xin_bytes=1 << 20, meta_elems=1 << 12), short: 4})
    if short == "xin_bytes":
        assert sess._capture[1].numel() == 16
    bufs = (sess.workspace, sess.k_cache, sess.v_cache, sess.dk_cache, sess.dv_cache, *sess._capture)
    torch.cuda.synchronize()
    before = [b.clone() for b in bufs]
    with pytest.raises(abi.AdtError) as e:
        sess.verify() if call == "verify" else sess.expand(1, 4, 16)
    assert e.value.code == abi.E_CAPACITY
    torch.cuda.synchronize()
    for b, was in zip(bufs, before):
        assert torch.equal(b.view(torch.uint8), was.view(torch.uint8))
    assert sess.captured() == []


def _normed(x):
    x = x.double()
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-5)


def test_fp32_view_shows_the_last_normed_activations(rt):
    """act in the view of an fp32 session: the RMSNorm of the residual rows that entered the last
    layer's MLP, after prompts (whose last forward is the draft's), expansions and verifies, and
    the same after a graph replay."""
    cfg, sess = _session(rt, "f32")
    d = cfg.model.d_model
    size = dict(resid_elems=1 << 20, xin_bytes=1 << 20, meta_elems=1 << 12)

    def act(rows):
        torch.cuda.synchronize()
        return sess._ws(sess.view().act, rows * d, torch.float32).view(rows, d).cpu()

    def check(what):
        rec = sess.captured()[-1]
        want = _normed(rec["resid"][-2])   # after the last layer's attention block
        got = act(rec["rows"])
        assert (got.double() - want).abs().max() <= 1e-5 * (1 + want.abs().max()), what
        sess.set_capture(0)
        return got

    sess.set_capture(**size)
    sess.prefill(synth.prefix_ids(cfg))
    check("prefill")
    for what, forward in (("expand", lambda: sess.expand(2, 3, 9)), ("verify", sess.verify)):
        sess.set_capture(**size)
        forward()
        got = check(what)
        sess._ws(sess.view().act, got.numel(), torch.float32).zero_()
        for _ in range(2):   # captured into a graph, then replayed
            forward()
        assert torch.equal(act(got.shape[0]), got), what


def test_failed_prefill_keeps_its_prompt(rt):
    """A prefill that fails after its prompt was queued for the device, behind work that is still
    running, has used that prompt and not the one of the call after it."""
    from paper_2512_21857_amd import abi
    cfg, sess = _session(rt, "f32")
    m = cfg.model
    first = synth.prefix_ids(cfg)
    second = first[::-1].copy()
    assert (first != second).any()
    # room for the target forward over the prompt, none for the draft's
    sess.set_capture(resid_elems=(2 * m.n_layers + 1) * cfg.prefix_len * m.d_model, xin_bytes=16, meta_elems=1 << 12)
    torch.cuda.synchronize()
    torch.cuda._sleep(100_000_000)
    for prompt in (first, second):
        with pytest.raises(abi.AdtError) as e:
            sess.prefill(prompt)
        assert e.value.code == abi.E_CAPACITY
    recs = sess.captured()
    assert len(recs) == 1 and recs[0]["tok"].tolist() == first.tolist()
