"""GPU parity of the vocabulary indexes behind the mask build (the vocabulary in byte order with
its two-byte prefix ranges, the byte-pair index), of the forced continuation of a Write run, and
of the sharing of cache keys between instances of one shape -- all through the C ABI, against the
CPU oracle, bit for bit."""
import numpy as np
import pytest

import wg_synth as ws
from oracle import oracle as O
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2507_16768_amd as wg
    wg.load_library()
    return torch


def _states_of_instances(o, n_inst):
    """(sid, description) of every state of the first n_inst template instances."""
    out = []
    for sid in range(1, o.num_states):
        d = o.describe(sid)
        if d["tmpl"] >= n_inst:
            break
        out.append((sid, d))
    return out


@pytest.mark.parametrize("idx,n_inst", [(2, 1), (3, 1), (4, 8), (5, 16)])
def test_every_literal_state_at_full_size(torch_cuda, idx, n_inst):
    """Every Write-byte state of the config at its full vocabulary (config 4: of its first eight
    instances): the mask equals the oracle's, and a state followed by another literal byte (or by
    the end) looks at the tokens sharing its two-byte prefix only.  In these vocabularies a quarter
    of the tokens that start with a byte are that byte alone (all of them allowed, so all of them
    looked at); of the tokens looked at in vain, at least nine in ten are gone compared with
    looking at every token that shares the first byte."""
    torch = torch_cuda
    w = ws.make_workload(idx, steps=1)
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    first_byte = np.zeros(256, dtype=np.int64)
    lens = np.diff(w.vocab.offsets.astype(np.int64))
    has = lens > 0
    np.add.at(first_byte, w.vocab.bytes[w.vocab.offsets[:-1][has].astype(np.int64)], 1)
    lit = [(sid, d) for sid, d in _states_of_instances(o, n_inst) if d["kind"] == "LIT"]
    assert len(lit) >= 10
    # (a) the states whose successor is a literal byte or takes no byte: candidates by prefix
    direct = [(sid, d) for sid, d in lit if o.describe(d["next"])["kind"] in ("LIT", "END")]
    deep = [(sid, d) for sid, d in lit if o.describe(d["next"])["kind"] not in ("LIT", "END")]
    for name, group in (("direct", direct), ("deep", deep)):
        for lo in range(0, len(group), 256):
            part = group[lo:lo + 256]
            print("cfg%d %s literal states %d..%d of %d" % (idx, name, lo, lo + len(part), len(group)), flush=True)
            st = np.array([[sid, 0] for sid, _ in part], dtype=np.uint32)
            d_mask = torch.empty((len(st), h.W), dtype=torch.int32, device="cuda")
            before = h.cache_stats()
            h.fill_masks(H.dev_states(st), d_mask)
            got = H.host_mask(d_mask)
            after = h.cache_stats()
            allowed = 0
            for i, (sid, d) in enumerate(part):
                want = o.mask_row((sid, 0))
                assert (got[i] == want).all(), (idx, sid, d)
                allowed += int(H.bits(want, w.vocab.V).sum())
            assert after["builds"] - before["builds"] == len(part)
            if name == "direct":
                walked = after["entries_walked"] - before["entries_walked"]
                bucket = int(sum(first_byte[d["byte"]] for _, d in part))
                assert allowed <= walked and (walked - allowed) * 10 <= bucket - allowed, (walked, allowed, bucket)
    assert len(direct) > 0


@pytest.mark.parametrize("V", [5003, 8193, 20011, 70001])
def test_the_candidates_counted_are_the_keys_own(torch_cuda, V):
    """entries_walked per made row: what the indexes hold for the key, counted here from the tokens' bytes, however many
    workgroups make the row (some of them without a token, where ranges are longer than shares)."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    vocab = ws.make_workload(4, V=V, B=1, steps=1).vocab
    text = 'Sequence(Wait(denies={}, wait={<}), Wait(allow={a, b}, wait={>}), Write("xyz"), Wait(denies={}, wait={<}))'
    toks = [bytes(vocab.bytes[int(a):int(b)]) for a, b in zip(vocab.offsets[:-1], vocab.offsets[1:])]
    two = sum(t == b"x" or t[:2] == b"xy" for t in toks), sum(t == b"y" or t[:2] == b"yz" for t in toks)
    want = {1: sum(t[:-1].count(b"<") for t in toks),                   # the exit leads to a checkpoint: every place of its byte but the last
            2: sum(t[:1] in (b"a", b"b", b">") and t != b"" for t in toks),   # few byte values enter: every token that begins with one
            3: two[0], 4: two[1],                                       # a literal in front of a literal: the byte itself, and the pair
            5: sum(t[:1] == b"z" for t in toks)}                        # a literal in front of a checkpoint
    h = wg.Handle([text], None, wg.Vocab(vocab.bytes, vocab.offsets, vocab.eos_id), flags=wg.EOS_RESTART)
    for sid, n in want.items():
        assert n > 0
        for B in (1, 3, 16, 64, 100, 256, 257, 700):
            st = H.dev_states(np.tile(np.array([[sid, 0]], dtype=np.uint32), (B, 1)))
            mask = torch.empty((B, h.W), dtype=torch.int32, device="cuda")
            h.cache_clear()
            before = h.cache_stats()["entries_walked"]
            h.fill_masks(st, mask)
            assert h.cache_stats()["entries_walked"] - before == B * n, (sid, B)


@pytest.mark.parametrize("idx,n_inst", [(2, 1), (3, 1), (4, 6), (5, 16)])
def test_every_checkpoint_state_at_full_size(torch_cuda, idx, n_inst):
    """Every Wait / condition state (all byte budgets that bind, for a bounded Wait) at the full
    vocabulary: whether its candidates come from the byte-pair index, by the exit byte or by the first byte."""
    torch = torch_cuda
    w = ws.make_workload(idx, steps=1)
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    lmax = w.vocab.lmax
    st = []
    for sid, d in _states_of_instances(o, n_inst):
        if d["kind"] in ("WAIT", "COND"):
            st.append([sid, 0])
            if d["kind"] == "WAIT" and d["max"] >= 0:
                st += [[sid, max(0, d["max"] - r)] for r in (0, 1, 2, 7, lmax - 1) if d["max"] - r >= 0]
    st = np.array(st, dtype=np.uint32)
    if idx == 5:
        st = st[::3]                                       # (several hundred states: every third)
    h.reserve_batch(len(st))
    d_mask = torch.empty((len(st), h.W), dtype=torch.int32, device="cuda")
    h.fill_masks(H.dev_states(st), d_mask)
    got = H.host_mask(d_mask)
    for i in range(len(st)):
        if i % 64 == 0:
            print("cfg%d checkpoint state %d of %d" % (idx, i, len(st)), flush=True)
        assert (got[i] == o.mask_row((int(st[i, 0]), int(st[i, 1])))).all(), (idx, st[i], o.describe(int(st[i, 0])))


@pytest.mark.parametrize("idx", [2, 3, 4, 5])
def test_forced_bytes_match_the_oracle(torch_cuda, idx):
    """wg_forced_bytes on every state of the config (plus ERROR, FINAL and out-of-range ids),
    with a roomy cap and with one that cuts the runs: bytes, lengths and end states."""
    torch = torch_cuda
    w = ws.make_workload(idx, steps=1)
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    sids = list(range(0, min(o.num_states, 6000))) + [O.SID_ERROR, o.num_states, o.num_states + 7]
    st = np.array([[s, (i * 7) % 5] for i, s in enumerate(sids)], dtype=np.uint32)
    d_states = H.dev_states(st)
    B = len(st)
    runs = 0
    for cap in (64, 3, 1):
        d_bytes = torch.full((B, cap), 0xEE, dtype=torch.uint8, device="cuda")
        d_lens = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        d_end = torch.full((B, 2), -1, dtype=torch.int32, device="cuda")
        h.forced_bytes(d_states, d_bytes, d_lens, d_end)
        gb, gl, ge = d_bytes.cpu().numpy(), d_lens.cpu().numpy(), H.host_states(d_end)
        for i, s in enumerate(sids):
            want, end = o.forced_bytes(s, cap)
            assert gl[i] == len(want) and bytes(gb[i, :gl[i]]) == want, (idx, s, cap)
            assert (gb[i, gl[i]:] == 0xEE).all()
            assert ge[i, 0] == end and ge[i, 1] == (0 if want else st[i, 1]), (idx, s, cap)
            runs += len(want) > 1
        h.forced_bytes(d_states, d_bytes, d_lens)            # end states are optional
        assert (d_lens.cpu().numpy() == gl).all()
    assert runs > 20
    assert (H.host_states(d_states) == st).all()             # the states are only read
    # feeding a forced run through wg_advance, byte by byte as single-byte tokens (ids 1..256 of
    # these vocabularies), leads to the reported end state
    lit = [s for s in sids[:400] if s < o.num_states and o.describe(s)["kind"] == "LIT"][:64]
    cur = np.array([[s, 0] for s in lit], dtype=np.uint32)
    d_cur = H.dev_states(cur)
    want = [o.forced_bytes(s, 64) for s in lit]
    for step in range(max(len(r) for r, _ in want)):
        tok = np.array([1 + r[step] if step < len(r) else -1 for r, _ in want], dtype=np.int32)
        keep = H.host_states(d_cur).copy()
        h.advance(d_cur, torch.from_numpy(np.where(tok < 0, 0, tok).astype(np.int32)).cuda())
        now = H.host_states(d_cur).copy()
        now[tok < 0] = keep[tok < 0]                         # (runs that have ended stay where they are)
        d_cur.copy_(H.dev_states(now))
    assert (H.host_states(d_cur)[:, 0] == np.array([e for _, e in want], dtype=np.uint32)).all()


def test_instances_of_one_shape_share_their_cache_rows(torch_cuda):
    """64 requests, each with its own instance of the same template and the same arguments: the
    global cache builds every distinct mask once, not once per instance, and the masks and
    states still equal the oracle's (whose instances know nothing of each other)."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    base = ws.make_workload(4, V=20011, B=2, steps=40)
    texts = [base.texts[i % 2] for i in range(64)]
    args = [base.args[i % 2] for i in range(64)]
    import dataclasses
    w = dataclasses.replace(base, texts=texts, args=args, B=64, request_template=np.arange(64, dtype=np.int64))
    one = dataclasses.replace(base)                          # one instance of each of the two shapes
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    st0 = H.start_states(o, w)
    assert (h.start_states[w.request_template] == st0).all()         # every instance keeps its own state ids
    assert h.cache_stats()["keys"] == wg.Handle(one.texts, one.args, v).cache_stats()["keys"]
    toks, sts, _ = o.trajectory(st0, w.token_draws(40))
    d_states = H.dev_states(st0)
    d_mask = torch.empty((64, h.W), dtype=torch.int32, device="cuda")
    cur = st0
    shapes_seen = set()
    for k in range(40):
        h.fill_masks(d_states, d_mask)
        assert (H.host_mask(d_mask) == o.fill_masks(cur)).all(), k
        for b in range(64):                                  # a mask is a function of (shape, state within it, budget)
            first = int(st0[b, 0])
            shapes_seen.add((b % 2, int(cur[b, 0]) - first, o.key_rem(tuple(cur[b]))))
        h.advance(d_states, torch.from_numpy(toks[k]).cuda())
        cur = sts[k]
        assert (H.host_states(d_states) == cur).all(), k
    s = h.cache_stats()
    assert s["builds"] == len(shapes_seen) and s["builds"] < 64 * 3, (s, len(shapes_seen))
    # a shape that joins later shares as well, a new shape gets keys of its own
    keys = s["keys"]
    h.add_instances(texts[:2], args[:2])
    assert h.cache_stats()["keys"] == keys
    other = ws.make_workload(4, V=20011, B=4, steps=1)
    h.add_instances(other.texts[2:3], other.args[2:3])
    assert h.cache_stats()["keys"] > keys


def test_two_live_handles_with_long_and_short_rows(torch_cuda):
    """A handle over the full 151,936-token vocabulary (19 KB rows, a share of them in each workgroup's
    LDS) stays usable after a handle over a 4,096-token vocabulary is compiled and used in the
    same process: fills of the two interleaved, every mask against the oracle."""
    torch = torch_cuda
    big = ws.make_workload(4, B=24, steps=4)
    small = ws.make_workload(2, V=4096, B=6, steps=4)
    ob = H.make_oracle(big)
    vb, hb = H.make_gpu(big)
    cur_b = H.start_states(ob, big)
    toks_b, sts_b, _ = ob.trajectory(cur_b, big.token_draws(4))
    os_ = H.make_oracle(small)
    vs, hs = H.make_gpu(small)                               # compiled after the long-row handle
    cur_s = H.start_states(os_, small)
    toks_s, sts_s, _ = os_.trajectory(cur_s, small.token_draws(4))
    d_b, d_s = H.dev_states(cur_b), H.dev_states(cur_s)
    m_b = torch.empty((big.B, hb.W), dtype=torch.int32, device="cuda")
    m_s = torch.empty((small.B, hs.W), dtype=torch.int32, device="cuda")
    for k in range(4):
        hs.fill_masks(d_s, m_s)
        hb.fill_masks(d_b, m_b)
        assert (H.host_mask(m_s) == os_.fill_masks(cur_s)).all(), k
        assert (H.host_mask(m_b) == ob.fill_masks(cur_b)).all(), k
        hb.advance(d_b, torch.from_numpy(toks_b[k]).cuda())
        hs.advance(d_s, torch.from_numpy(toks_s[k]).cuda())
        cur_b, cur_s = sts_b[k], sts_s[k]
    assert hb.error_count() == 0 and hs.error_count() == 0


@pytest.mark.timeout(600)
def test_cold_steps_at_full_size_from_the_middle_of_the_trajectory(torch_cuda):
    """The mode the benchmark times: config 4 at B=256, V=151,936, the cache cleared before every
    fill, on ten steps taken from the middle of the oracle's trajectory: the full [256, 4748]
    bitmask, the masked bf16 logits and the next states of every step."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    k_first, n = 200, 10                                  # (the oracle needs half a minute to get there)
    w = ws.make_workload(4, steps=k_first + n)
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    st0 = H.start_states(o, w)
    toks, sts, _ = o.trajectory(st0, w.token_draws(k_first + n))
    cur = sts[k_first - 1]
    d_states = H.dev_states(cur)
    d_mask = torch.empty((w.B, h.W), dtype=torch.int32, device="cuda")
    seen = {}
    for k in range(k_first, k_first + n):
        print("cold step %d" % k, flush=True)
        h.cache_clear()
        d_mask.fill_(0x2B2B2B2B)
        h.fill_masks(d_states, d_mask)
        got = H.host_mask(d_mask)
        for b in range(w.B):
            key = (int(cur[b, 0]), int(cur[b, 1]))
            if key not in seen:
                seen[key] = o.mask_row(key)
            assert (got[b] == seen[key]).all(), (k, b, key)
        host = H.logits_for(w, tag=k)
        d_log = H.dev_logits(host)
        wg.apply_mask(d_log, d_mask)
        want = O.apply_mask(host.copy(), got)
        assert (H.host_logit_bits(d_log) == want).all(), k
        h.advance(d_states, torch.from_numpy(toks[k]).cuda())
        cur = sts[k]
        assert (H.host_states(d_states) == cur).all(), k
    s = h.cache_stats()
    assert s["hits"] == 0 and s["lookups"] == n * w.B and h.error_count() == 0
    # the same through the single call, again cold on every step
    cur = sts[k_first - 1]
    d_states = H.dev_states(sts[k_first - 2])
    prev = torch.from_numpy(toks[k_first - 1]).cuda()
    for k in range(k_first, k_first + 4):
        print("cold decode_step %d" % k, flush=True)
        h.cache_clear()
        host = H.logits_for(w, tag=k)
        d_log = H.dev_logits(host)
        h.decode_step(d_states, prev, d_mask, d_log)
        assert (H.host_states(d_states) == cur).all(), k
        want_mask = np.stack([seen[(int(s_[0]), int(s_[1]))] for s_ in cur])
        assert (H.host_mask(d_mask) == want_mask).all(), k
        assert (H.host_logit_bits(d_log) == O.apply_mask(host.copy(), want_mask)).all(), k
        prev = torch.from_numpy(toks[k]).cuda()
        cur = sts[k]


def test_every_kind_of_class_table_and_candidate_source(torch_cuda):
    """Checkpoints chosen so that both ways to take a class table (by first byte, by token rows) and
    every candidate source of the row build are taken: printable text up to '<', a free-text Wait,
    allow lists; exits of one, six, seven and ten byte values in front of a literal (byte pairs), in
    front of the end, and in front of another checkpoint (places behind the exit byte); with and
    without byte budgets.  Every state and budget against the oracle on a 20,011-token vocabulary,
    cold and again warm."""
    torch = torch_cuda
    base = ws.make_workload(2, V=20011, B=1, steps=1)
    texts = [
        r'Sequence(Wait(allow={[\x20-\x7e]}, wait={<}), Write("/p>"), Wait(allow={[\x20-\x7e]}, wait={<}, max=9), Write("a"))',
        r'Sequence(Wait(allow={\w}, wait={\d}), Write("ab"), Wait(allow={\w, \s, \., -}, wait={\d}, max=5), Write("0"))',
        r'Sequence(Wait(denies={}, wait={a, b, c, d, e, f}), Write("gh"), Wait(denies={\n}, wait={a, b, c, d, e, f, g}), Write("hi"))',
        r'Sequence(Wait(allow={[a-z]}, wait={\d}), Wait(denies={}, wait={[0-4]}, max=12), Wait(allow={\d}, wait={;}))',
        r'IfElse(condition=Wait(allow={\ }, true_waits={[0-6]}, false_waits={[a-f]}), if_body=Write("x1"), else_body=None)',
        r'DoWhile(body=Sequence(Write("k"), Wait(allow={[\x20-\x7e]}, wait={\", \x27})), '
        r'condition=Wait(allow={\s}, true_waits={\,, ;}, false_waits={\., !, ?}))',
        r'Sequence(Write("q"), Wait(allow={[\x00-\xff]}, wait={<eos>}))',
    ]
    import dataclasses
    w = dataclasses.replace(base, texts=texts, args=[{}] * len(texts), B=len(texts),
                            request_template=np.arange(len(texts), dtype=np.int64))
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    lmax = w.vocab.lmax
    st = []
    for sid in range(1, o.num_states):
        d = o.describe(sid)
        st.append([sid, 0])
        if d["kind"] == "WAIT" and d["max"] >= 0:
            st += [[sid, a] for a in range(1, d["max"] + 2)]
    st = np.array(st, dtype=np.uint32)
    want = o.fill_masks(st)
    d_mask = torch.empty((len(st), h.W), dtype=torch.int32, device="cuda")
    for rep in ("cold", "warm"):
        d_mask.fill_(0x66666666)
        h.fill_masks(H.dev_states(st), d_mask)
        got = H.host_mask(d_mask)
        bad = np.nonzero((got != want).any(axis=1))[0]
        assert len(bad) == 0, (rep, st[bad[0]], o.describe(int(st[bad[0], 0])))
    s = h.cache_stats()
    assert s["class_scans"] >= 10 and s["hits"] == len(st)
    # and the advance of every token from the start state of each template
    V = w.vocab.V
    for t in range(len(texts)):
        s0 = o.start_state(t)
        rep_states = np.tile(np.array([[s0, 0]], dtype=np.uint32), (V, 1))
        tk = np.arange(V, dtype=np.int32)
        d_st = H.dev_states(rep_states)
        h.advance(d_st, torch.from_numpy(tk).cuda())
        assert (H.host_states(d_st) == o.advance(rep_states, tk)).all(), t


@pytest.mark.parametrize("tables", [0, 1, 2, 3, 8])
def test_many_class_tables_in_one_call(torch_cuda, tables):
    """Calls that bring 19 templates' class tables at once on a 20,011-token vocabulary (the last token
    range ragged): tables under which nearly every token leaves early, printable text up to one byte,
    free text, allow lists, a table no byte leaves.  Every state and budget against the oracle,
    cold, then cold again after a clear, then warm; then the same on a vocabulary of 5,000 tokens
    longer than 8 bytes that all leave their checkpoint after the eighth byte, on a vocabulary with
    tokens of up to 40 bytes, and on every state of a reduced config 5.  wg_set_scan_batch takes 0 to 8
    and changes nothing."""
    torch = torch_cuda
    base = ws.make_workload(2, V=20011, B=1, steps=1)
    texts = []
    for i in range(8):        # one allowed letter, every other printable byte leaves: a candidate per place in a token
        a = chr(ord("a") + i)
        texts.append(r'Sequence(Wait(allow={%s}, wait={[\x20-\x60], [\x7b-\x7e], %s}), Write("%s."))'
                     % (a, ", ".join(chr(c) for c in range(ord("a"), ord("z") + 1) if chr(c) != a), a))
    for i in range(6):        # printable text up to one byte
        texts.append(r'Sequence(Wait(allow={[\x20-\x7e]}, wait={%s}, max=%d), Write("ok"))'
                     % (("<", ">", r"\x7b", r"\x7d", r"\x5b", r"\x5d")[i], 3 + i))
    texts += [
        r'Sequence(Wait(denies={}, wait={\n}), Write("x"))',
        r'Sequence(Wait(allow={\d}, wait={;}), Wait(allow={[a-f]}, wait={\,}, max=4))',
        r'Sequence(Write("q"), Wait(allow={[\x00-\xff]}, wait={<eos>}))',
        r'IfElse(condition=Wait(allow={\s}, true_waits={[0-6]}, false_waits={[a-f]}), if_body=Write("x1"), else_body=None)',
        r'DoWhile(body=Write("k"), condition=Wait(allow={\ }, true_waits={\,}, false_waits={\.}))',
    ]
    import dataclasses
    w = dataclasses.replace(base, texts=texts, args=[{}] * len(texts), B=len(texts),
                            request_template=np.arange(len(texts), dtype=np.int64))

    def every_state(o):
        st = []
        for sid in range(1, o.num_states):
            d = o.describe(sid)
            st.append([sid, 0])
            if d["kind"] == "WAIT" and d["max"] >= 0:
                st += [[sid, a] for a in range(1, d["max"] + 2)]
        return np.array(st, dtype=np.uint32)

    # long tokens: 8 to 15 letters a, then b, then a tail; under a table that lets a stay and leaves
    # at b, the first 8 bytes decide none of them, so every walk goes on into the next chunk and
    # from there into the successor
    from wg_synth.vocab import from_tokens
    long_tokens = [b""] + [bytes([x]) for x in b"abcdefgh<."]
    for i in range(5000):
        tail = bytes(ord("c") + (i // 24 ** k) % 24 for k in range(3))      # i in base 24: no two alike
        long_tokens.append(b"a" * (8 + i % 8) + b"b" + tail)
        if i % 5 == 0:
            long_tokens.append(b"a" * (1 + i % 4) + b"b" + tail)            # short ones between them
    long_texts = [r'Sequence(Wait(allow={a, %s}, wait={b}), Wait(allow={[c-z]}, wait={.}))' % chr(ord("c") + i)
                  for i in range(9)]                 # every tail is allowed behind the b: a lost candidate is a lost token
    long_w = dataclasses.replace(base, vocab=from_tokens(long_tokens, eos_id=0), texts=long_texts, args=[{}] * len(long_texts),
                                 B=len(long_texts), request_template=np.arange(len(long_texts), dtype=np.int64))
    assert len(set(long_tokens)) == len(long_tokens) and long_w.vocab.lmax <= 24

    # tokens of up to 40 bytes: longer than the 24 bytes of a run that a walk holds
    wide = ws.make_vocab(3001, ("geometric", 10, 40), seed=9, utf8_tenths=1)
    assert wide.lmax == 40
    wide_w = dataclasses.replace(ws.make_workload(5, V=3001, B=16, steps=1), vocab=wide)

    for label, wl in (("chosen", w), ("long tokens", long_w), ("tokens up to 40 bytes", wide_w),
                      ("config 5", ws.make_workload(5, V=7013, B=16, steps=1))):
        print(label, tables, flush=True)
        o = H.make_oracle(wl)
        v, h = H.make_gpu(wl)
        h.set_scan_batch(tables)
        st = every_state(o)
        h.reserve_batch(len(st))
        want = o.fill_masks(st)
        d_mask = torch.empty((len(st), h.W), dtype=torch.int32, device="cuda")
        for rep in ("cold", "cleared", "warm"):
            if rep == "cleared":
                h.cache_clear()
            d_mask.fill_(0x66666666)
            h.fill_masks(H.dev_states(st), d_mask)
            got = H.host_mask(d_mask)
            bad = np.nonzero((got != want).any(axis=1))[0]
            assert len(bad) == 0, (label, rep, st[bad[0]], o.describe(int(st[bad[0], 0])))
        s = h.cache_stats()
        assert s["class_scans"] >= {"chosen": 38, "long tokens": 18}.get(label, 20) and s["hits"] == len(st), s
        assert h.error_count() == 0
    with pytest.raises(Exception):
        h.set_scan_batch(9)


@pytest.mark.timeout(600)
def test_the_largest_batch_one_call_takes(torch_cuda):
    """B = 65,535 requests in one call (the most a call takes; one more is refused): masks, masked
    fp32 logits and next states of every request, the requests spread over every state of a
    config-3 instance on a 1,003-token vocabulary."""
    torch = torch_cuda
    import paper_2507_16768_amd as wg
    B = 65535
    w = ws.make_workload(3, V=1003, B=4, steps=1)
    o = H.make_oracle(w)
    v, h = H.make_gpu(w)
    with pytest.raises(wg.WgError):
        h.reserve_batch(B + 1)
    h.reserve_batch(B)
    distinct = []
    for sid in range(0, o.num_states):
        d = o.describe(sid)
        distinct.append((sid, 0))
        if d["kind"] == "WAIT" and d["max"] >= 0:
            distinct += [(sid, d["max"] - r) for r in range(0, 12) if d["max"] - r > 0]
    distinct.append((O.SID_ERROR, 0))
    rows = np.stack([o.mask_row(s) for s in distinct])
    pick = (np.arange(B) * 7919) % len(distinct)
    st = np.array([distinct[i] for i in pick], dtype=np.uint32)
    d_states = H.dev_states(st)
    d_mask = torch.full((B, h.W), 0x0F0F0F0F, dtype=torch.int32, device="cuda")
    h.fill_masks(d_states, d_mask)
    assert (H.host_mask(d_mask) == rows[pick]).all()
    s = h.cache_stats()
    assert s["lookups"] == B and s["builds"] == len({(sid, o.key_rem((sid, aux))) for sid, aux in distinct if sid != O.SID_ERROR})
    # masked logits: the same 1,003 values in every row, so that the expectation stays small
    x = ws.make_logits(5, 1, w.vocab.V, 1.0)
    d_log = torch.from_numpy(np.repeat(x, B, axis=0)).cuda()
    wg.apply_mask(d_log, d_mask)
    want_rows = np.stack([O.apply_mask(x.copy(), rows[i:i + 1])[0] for i in range(len(distinct))]).view(np.uint32)
    assert (H.host_logit_bits(d_log) == want_rows[pick]).all()
    # next states: every request takes the first token its mask allows (or token 1 where none is)
    tok_of = np.array([O.select_bit(r, 0) if r.any() else 1 for r in rows], dtype=np.int32)
    toks = tok_of[pick]
    h.advance(d_states, torch.from_numpy(toks).cuda())
    nxt = o.advance(np.array(distinct, dtype=np.uint32), tok_of)
    assert (H.host_states(d_states) == nxt[pick]).all()
    # and the whole step in one call, with the cache cleared
    d_states2 = H.dev_states(st)
    h.cache_clear()
    d_log2 = torch.from_numpy(np.repeat(x, B, axis=0)).cuda()
    d_mask.fill_(0)
    h.decode_step(d_states2, None, d_mask, d_log2)
    assert (H.host_mask(d_mask) == rows[pick]).all()
    assert (H.host_logit_bits(d_log2) == want_rows[pick]).all()
