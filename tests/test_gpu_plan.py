"""The bulk append's plan, and the plan of a decode call of many sequences, at
the sizes where they split differently: around one token per lane and round,
around a whole chunk of tokens and across chunks, with a recent window, with a
pool that runs out inside a chunk, and with the online controller near its
reserves.  Decisions, slots, counters, lists and
budgets against the CPU oracle, all exact."""

import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import Scenario, budgets, say
from workload import make_policy
from workload.tags import function_call_tags
from workload.policy import PolicyTable, contiguous_groups, pack_blob

pytestmark = pytest.mark.gpu

H, D = 1, 64


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_28276_amd.pask  # noqa: F401  (fails loudly when libpask.so is missing)


def _session(pol, B, L, max_tok, hi=None, lo=None):
    from paper_2608_28276_amd.session import PaskSession
    pages = B * L * ((max_tok + 15) // 16 + 1)
    return PaskSession(pack_blob(pol), max_batch=B, n_layers=L, n_q_heads=H, n_kv_heads=H, head_dim=D,
                       max_tokens_per_seq=max_tok, hi_pages=hi or pages, lo_pages=lo or pages)


def _check_lists(sess, b, layer, acts, what):
    """Stores of (b, layer) against the actions of positions 0.. that were persisted."""
    hi, lo = oracle.compact(acts, np.arange(acts.size))
    cnt = sess.counters()[b, layer].cpu().numpy()
    assert (int(cnt[0]), int(cnt[1]), int(cnt[3])) == (hi.size, lo.size, int((acts == oracle.DROP).sum())), (what, cnt)
    il = sess.index_lists()[b, layer].cpu().numpy()
    assert (il[0, :hi.size] == hi).all() and (il[1, :lo.size] == lo).all(), what
    bt = sess.block_tables()[b, layer].cpu().numpy()
    for st, n in ((0, hi.size), (1, lo.size)):
        used = bt[st, :(n + 15) // 16]
        assert np.unique(used).size == used.size, (what, "a page twice in one store")


@pytest.mark.parametrize("W", [0, 37])
@pytest.mark.parametrize("n", [63, 64, 65, 1023, 1024, 1025, 2049, 16383, 16384, 16385, 33000])
def test_bulk_plan_sizes(n, W):
    """Three sequences take n, n // 3 and 1 tokens, then all take 65 more."""
    say(f"case: plan n={n} W={W}")
    pol = make_policy(6, 1, 1, 0.4, 3, n_sink=5)
    pol.recent_window = W
    B, more = 3, 65
    sess = _session(pol, B, 1, n + more)
    rng = np.random.default_rng(n)
    counts = np.array([n, n // 3, 1], np.int32)
    tags = [rng.integers(0, 6, (B, m)).astype(np.uint8) for m in (n, more)]
    put = lambda x: torch.as_tensor(x, device=sess.device)
    k, k2 = (torch.ones((B, m, H, D), dtype=torch.bfloat16, device=sess.device) for m in (n, more))
    sess.append(0, put(tags[0]), k, k, n_new=put(counts))
    sess.append(0, put(tags[1]), k2, k2)
    for b in range(B):
        z = np.concatenate([tags[0][b, :counts[b]], tags[1][b]])
        acts, _, _ = oracle.decide(z, np.arange(z.size), 0, pol.action, pol.floor, pol.n_sink, False)
        _check_lists(sess, b, 0, acts[:max(0, z.size - W)], (n, W, b))
        assert int(sess.counters()[b, 0, 2]) == z.size


@pytest.mark.parametrize("W", [0, 5])
@pytest.mark.parametrize("n", [1, 2, 40, 1025])
@pytest.mark.parametrize("keep_all", [True, False])
def test_tags_outside_the_table_are_reported(n, W, keep_all):
    """A tag outside the table raises BAD_TAG however many tokens the call has,
    whether the tokens are kept by their tags or all of them; a bad tag past
    n_new, or past the sequence's capacity, is none."""
    from paper_2608_28276_amd import pask
    say(f"case: bad tag n={n} W={W} keep_all={keep_all}")
    pol = make_policy(6, 1, 1, 0.4, 3)
    pol.recent_window = W
    room = 8                                         # the window fits the shortest sequence
    put = lambda x: torch.as_tensor(x, device="cuda:0")
    for z, at in ((5, n - 1), (6, n - 1), (255, 0), (6, n)):
        sess = _session(pol, 1, 1, n + room)
        tags = np.zeros((1, n + 1), np.uint8)
        tags[0, at] = z
        k = torch.ones((1, n + 1, H, D), dtype=torch.bfloat16, device=sess.device)
        if at < n and n == 1:                        # one token: also the call without n_new
            sess.append(0, put(tags[:, :1].copy()), k[:, :1].contiguous(), k[:, :1].contiguous(), keep_all=keep_all)
        else:
            sess.append(0, put(tags), k, k, n_new=put(np.array([n], np.int32)), keep_all=keep_all)
        _, _, bad = oracle.decide(tags[0, :n], np.arange(n), 0, pol.action, pol.floor, pol.n_sink, keep_all)
        assert sess.stats(batch=1)[0].device_flags == (pask.PASK_FLAG_BAD_TAG if bad.any() else 0), (z, at)
        cnt = sess.counters()[0, 0].cpu().numpy()
        assert int(cnt[2]) == n
        if keep_all:
            assert int(cnt[0]) == max(0, n - W)
    sess = _session(pol, 1, 1, 30)                   # a bad tag of a token there is no room for
    tags = np.zeros((1, 40), np.uint8)
    tags[0, 35] = 77
    k = torch.ones((1, 40, H, D), dtype=torch.bfloat16, device=sess.device)
    if n == 40:
        with pytest.raises(Exception):
            sess.append(0, put(tags), k, k, keep_all=keep_all)   # more than a sequence holds: refused
        sess.append(0, put(tags[:, :20].copy()), k[:, :20].contiguous(), k[:, :20].contiguous(), keep_all=keep_all)
        sess.append(0, put(tags[:, 20:].copy()), k[:, 20:].contiguous(), k[:, 20:].contiguous(), keep_all=keep_all)
        assert sess.stats(batch=1)[0].device_flags == pask.PASK_FLAG_SEQ_CAPACITY


@pytest.mark.parametrize("pages", [3, 64, 1100])
def test_pool_runs_out_inside_a_chunk(pages):
    """20,000 HIGH tokens of one sequence and room for `pages` pages: the first
    16 * pages tokens are stored, the rest counted as lost and flagged."""
    from paper_2608_28276_amd import pask
    say(f"case: plan, HIGH pool of {pages} pages")
    n = 20000
    pol = make_policy(6, 1, 1, 0.4, 3)
    sess = _session(pol, 1, 1, n, hi=pages)
    k = torch.ones((1, n, H, D), dtype=torch.bfloat16, device=sess.device)
    sess.append(0, None, k, k, keep_all=True)
    cnt = sess.counters()[0, 0].cpu().numpy()
    assert (cnt[:6] == [16 * pages, 0, n, 0, 16 * pages, n - 16 * pages]).all(), cnt
    assert (sess.index_lists()[0, 0, 0, :16 * pages].cpu().numpy() == np.arange(16 * pages)).all()
    st, status, _ = sess.stats(batch=1)
    assert status == pask.PASK_E_DEVICE_FLAG and st.device_flags == pask.PASK_FLAG_HI_POOL_EXHAUSTED


@pytest.mark.parametrize("seed", [0, 1, 2])
@pytest.mark.parametrize("n", [200, 1500])
def test_controller_near_its_reserves(n, seed):
    """Five groups of one to three layers under random tables, scores (ties and
    zeros among them), reserves spread over the whole budget and iid parser
    states, so that runs are cut at every kind of token: unconstrained, partly
    demoted, partly promoted, at the floors, sinks, unknown tags and states."""
    say(f"case: controller plan n={n} seed={seed}")
    rng = np.random.default_rng(seed)
    C, T, S = 5, 7, 40
    gol = np.repeat(np.arange(C), [1, 3, 2, 1, 2]).astype(np.uint8)
    L = gol.size
    pol = PolicyTable(n_tags=T, n_groups=C, n_layers=L, group_of_layer=gol,
                      action=rng.integers(0, 3, (T, C)).astype(np.uint8),
                      floor=(rng.integers(0, 3, (T, C)) * (rng.random((T, C)) < 0.3)).astype(np.uint8),
                      rho_up=rng.integers(0, 4, (T, C, 2)).astype(np.float32), n_sink=3)
    pol.n_states, pol.beta_q = S, 65536 // 3
    pol.reserve_q = (16 * n / 3 * rng.random(S) * (rng.random(S) < 0.9)).astype(np.uint32)
    pol.crit = (rng.random(S) < 0.5).astype(np.uint8)
    B = 2
    sess = _session(pol, B, L, n)
    sess.budget_init(n, batch=B)
    tags = rng.integers(0, T + 1, (B, n)).astype(np.uint8)
    tags[:, :] = np.where(rng.random((B, n)) < 0.97, tags % T, tags)
    states = rng.integers(0, S + 1, (B, n)).astype(np.uint8)
    k = torch.ones((B, n, H, D), dtype=torch.bfloat16, device=sess.device)
    put = lambda x: torch.as_tensor(np.ascontiguousarray(x), device=sess.device)
    cut = n // 2 + 13
    m = oracle.group_costs(gol, C, H, D)
    gamma = oracle.reserve_bytes(pol.reserve_q, m)
    for layer in range(L):
        for j0, j1 in ((0, cut), (cut, n)):
            sess.append(layer, put(tags[:, j0:j1]), k[:, j0:j1].contiguous(), k[:, j0:j1].contiguous(),
                        states=put(states[:, j0:j1]))
    R_gpu = budgets(sess.counters().cpu().numpy())
    kinds = set()
    for b in range(B):
        R = oracle.initial_budget(pol.beta_q, n, m)
        acts = np.zeros((n, C), np.uint8)
        for i in range(n):
            z, s = int(tags[b, i]), int(states[b, i])
            known = s < S
            forced = i < 3 or z >= T
            acts[i], cost = oracle.online_actions(z, s, R, pol.action, pol.floor, pol.rho_up, m,
                                                  gamma[s] if known else 0, bool(pol.crit[s]) if known else False,
                                                  forced)
            if not forced:
                a0 = np.maximum(pol.action[z], pol.floor[z])
                kinds.add((bool((acts[i] < a0).any()), bool((acts[i] > a0).any()),
                           bool((acts[i] == pol.floor[z]).all())))
            R -= cost
        assert (R_gpu[b] == R).all(), (b, R_gpu[b], R)
        for layer in range(L):
            _check_lists(sess, b, layer, acts[:, gol[layer]], (n, seed, b, layer))
    assert len(kinds) >= 3, kinds


@pytest.mark.parametrize("B", [65, 320, 1024, 1025])
def test_decode_call_of_many_sequences(B):
    """A decode call that persists its tokens plans 64 sequences per wave and
    pass, up to 1,024 of them; above, the one-token append comes first and the
    plan reads the counters past the 1,024th.  Short ragged prompts, some
    empty, so that pages open in every chunk; two steps, all compared."""
    say(f"case: decode plan of {B} sequences")
    pol = make_policy(6, 1, 1, 0.4, seed=B)
    P = [(7 * b) % 35 for b in range(B)]
    base = function_call_tags(B + 2, 5)
    tags = np.stack([base[b:b + 2] for b in range(B)])
    sc = Scenario(pol, B=B, L=1, Hq=2, Hkv=1, D=64, prompt_lens=P, gen_tags=tags, seed=B)
    sc.fill_prompt()
    for t in range(2):
        sc.decode_step(t)
    sc.check_state()


@pytest.mark.parametrize("B,Hkv,D", [(16, 8, 128), (17, 8, 128), (18, 7, 64), (64, 2, 64), (64, 3, 64)])
def test_decode_call_around_few_segments(B, Hkv, D):
    """128 (sequence, KV head) segments and fewer are cut one by one, more as
    ranges over the whole list, here by every worker (short histories): lengths
    from 0 to 70 pages, so that segments have one to several pieces, and one
    sequence of 1,900 tokens; both stores; two steps."""
    say(f"case: decode of {B} x {Hkv} segments, D={D}")
    P = [(97 * b) % 1100 for b in range(B)]
    P[-1] = 1900
    _two_steps(B, Hkv, D, P)


@pytest.mark.parametrize("B,Hkv,D", [(17, 8, 128), (33, 4, 128), (19, 7, 64), (65, 2, 64), (130, 1, 64)])
def test_decode_call_of_long_histories(B, Hkv, D):
    """More than 128 segments whose history is long (64 pages a sequence and
    more) and mostly HIGH are streamed by few workers, the first wave or two of
    each workgroup: lengths of 1,100 to 2,900 tokens, some sequences empty or of
    one page; both stores; two steps."""
    say(f"case: decode of {B} x {Hkv} long segments, D={D}")
    P = [1100 + (397 * b) % 1800 for b in range(B)]
    P[1], P[B // 2] = 0, 9
    counts = np.asarray(P) + 40
    assert np.sum(counts // 16) >= 64 * B and 40 * B < counts.sum() / 6, "few workers"
    _two_steps(B, Hkv, D, P)


def _two_steps(B, Hkv, D, P):
    pol = make_policy(6, 1, 1, 0.4, seed=B + Hkv)
    base = function_call_tags(B + 40, 6)
    tags = np.stack([base[b:b + 40] for b in range(B)])
    sc = Scenario(pol, B=B, L=1, Hq=2 * Hkv, Hkv=Hkv, D=D, prompt_lens=P, gen_tags=tags, seed=B)
    sc.fill_prompt()
    sc.append_steps(0, 38)
    sc.decode_step(38)
    sc.decode_step(39)
    sc.check_state()


@pytest.mark.parametrize("G", [1, 4, 8])
@pytest.mark.parametrize("n", [900, 17000])
def test_merge_of_many_pieces(n, G):
    """One sequence of few KV heads and many pages: the merge of the fewest
    segments folds 64 pieces per round (17,000 tokens: more than one round)."""
    say(f"case: merge of many pieces, n={n} G={G}")
    pol = make_policy(6, 1, 1, 0.4, seed=G)
    sc = Scenario(pol, B=1, L=1, Hq=2 * G, Hkv=2, D=64 if G == 1 else 128, prompt_lens=[n],
                  gen_tags=function_call_tags(3, 9)[None], seed=n + G, max_ctx_hint=n + 600)
    sc.fill_prompt()
    for t in range(3):
        sc.decode_step(t)
    sc.check_state()
