"""A session's forwards where their bookkeeping ends."""
import dataclasses

import numpy as np
import pytest
import torch

import synth
from oracle.tree import ancestors_and_self, depths

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


class _ForcedImage:
    """A configuration whose every image cell allows one id, so that an image of any length can be
    committed by chains of the ids it must have."""

    def __init__(self, cfg, ids):
        self._cfg, self.ids = cfg, ids

    def __getattr__(self, name):
        return getattr(self._cfg, name)

    def allowed_table(self):
        return np.stack([self.ids, self.ids + 1], axis=1).astype(np.int32)


def _fragment_rows(att, rows, d):
    """The rows of a buffer in the layout of the projections' inputs (documented at the view)."""
    B = (rows + 15) // 16
    r, k = torch.arange(rows, device=att.device)[:, None], torch.arange(d, device=att.device)[None, :]
    return att[(((k // 32) * B + r // 16) * 64 + r % 16 + 16 * ((k % 32) // 8)) * 8 + k % 8]


@pytest.mark.parametrize("head_dim,heads,guided", [(64, 20, False), (128, 20, False), (64, 4, True), (128, 4, False)])
def test_session_attention_merges_many_key_splits(rt, head_dim, heads, guided):
    """One session from the start of a 2352-cell image to its end: at four prefix lengths, trees
    of every tile count are verified and the layer's attention output is compared with 64 bits over
    the session's own queries and caches.  The keys have ten splits at the cache's capacity, of
    which one or two, two to five, six to eight and nine or ten hold keys (past eight, the merge
    takes a second pass), so one set of arrival counters serves growing numbers of splits.  Twenty
    heads merge in the attention's launch up to 64 rows of head size 64 and 16 of 128, four
    up to 32 and 8; trees with more rows do so while one split holds all their keys, and then in
    a launch of its own.  A repeated verify gives the same bits.

    The kernel rounds each unnormalised probability and the output to bf16, at most 2^-9 of
    each value; over a row of independent values that is at most 2^-8 of its 2-norm
    (the fp32 sums add about 1e-6).  Losing one split of ten would be about 0.3."""
    nb = 2 if guided else 1
    cfg = synth.shrink(synth.get_config("lumina_7b"), n_layers=1, d_model=heads * head_dim, n_heads=heads, head_dim=head_dim,
                       ffn=256, vocab=1024)
    sched = dataclasses.replace(cfg.sched, d_lo=1, d_hi=30, k_lo=1, k_hi=4, alpha_source="real")
    cfg = dataclasses.replace(cfg, prefix_len=60, prefix_lo=0, prefix_hi=1024, img_lo=0, img_hi=1024, row_end_col=-1,
                              grid_w=49, sched=sched, guidance=3.0 if guided else None)
    if guided:
        cfg = dataclasses.replace(cfg, sched=dataclasses.replace(sched, n_budget=40))
    P, m = cfg.prefix_len, cfg.model
    rng = np.random.default_rng([head_dim, nb])
    img = _ForcedImage(cfg, rng.integers(0, 1024, size=cfg.n_image).astype(np.int32))
    sess = rt.DeviceSession(rt.DeviceModel(cfg, synth.model_weights(cfg)), img)
    assert sess.prefill(synth.prefix_ids(cfg), synth.null_prefix_ids(cfg) if guided else None) == img.ids[0]
    for target in (P, 440, 1300, 2290):
        while sess.view().L < target:
            v = sess.view()
            g = v.L - P   # the image cell of the root
            chain = min(31, target - v.L, cfg.n_image - g)
            sess.expand(1, 1, 1)   # keeps the draft cache up with the commits
            sess.set_tree([-1] + list(range(chain - 1)), img.ids[g: g + chain])
            sess.verify()
            assert sess.accept_commit(1, 1)["n_accepted"] == chain - 1
        L = sess.view().L
        for cache in (sess.k_cache, sess.v_cache):   # keys and values of every size, not the small model's
            cache.normal_(generator=torch.Generator(device="cuda").manual_seed(L))
        for n in (1, 11, 17, 33, 64) if guided else (1, 8, 11, 17, 32, 40, 61, 100, 128):
            if L + n > sess.s_cap:
                continue
            parent = synth.random_parents(rng, n, max_depth=8)
            order = np.argsort(depths(parent), kind="stable")
            inv = np.argsort(order)
            parent = np.array([-1 if parent[o] < 0 else inv[parent[o]] for o in order], dtype=np.int32)
            token = rng.integers(0, 1024, size=n).astype(np.int32)
            token[0] = img.ids[L - P]
            sess.set_tree(parent, token)
            see = torch.zeros(n, L + n, dtype=torch.bool, device="cuda")
            see[:, :L] = True
            for i, anc in enumerate(ancestors_and_self(parent)):
                see[i, [L + j for j in anc]] = True
            first = None
            for _ in range(3):
                sess.verify()
                v = sess.view()
                att = _fragment_rows(sess._ws(v.att, (nb * n + 15) // 16 * 16 * m.d_model, torch.bfloat16), nb * n,
                                     m.d_model).clone()
                first = att if first is None else first
                assert torch.equal(att, first), (L, n)
            q = sess._ws(v.q, nb * n * m.d_model, torch.bfloat16).view(n, nb, m.n_heads, head_dim).double()
            got = first.view(n, nb, m.n_heads, head_dim).double()
            for b in range(nb):
                k, vv = ((c[b, 0] if guided else c[0])[:, : L + n].double() for c in (sess.k_cache, sess.v_cache))
                s = torch.matmul(q[:, b].transpose(0, 1).contiguous(), k.transpose(1, 2).contiguous()) / head_dim ** 0.5
                p = torch.softmax(s.masked_fill(~see, float("-inf")), -1)
                ref = torch.matmul(p, vv.contiguous()).transpose(0, 1)
                rel = (got[:, b] - ref).norm(dim=-1) / ref.norm(dim=-1)
                assert rel.max() <= 2.0 ** -7, (L, n, b, rel.max().item())
