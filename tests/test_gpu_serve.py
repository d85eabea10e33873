"""GPU parity of the serving-step entry points: verification attention over a
paged KV cache, target argmax + acceptance from logits, and the KV commit of
the accepted path -- against the oracle (and the contiguous GPU path)."""
import sys

import numpy as np
import pytest

import oracle
import synth
from tests import gpu_common as gc

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu():
    gc.require_gpu()


def _log(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def to_pages(k_cache, v_cache, kv_offsets, page_size, rng, spare=2):
    """Scatter each request's prefix into shuffled pages; returns
    (k_pages, v_pages, block_table, prefix_len)."""
    R = len(kv_offsets) - 1
    P = np.diff(kv_offsets).astype(np.int64)
    npg = (P + page_size - 1) // page_size
    maxp = int(npg.max()) + spare
    total = int(npg.sum()) + spare * R
    perm = rng.permutation(total).astype(np.int32)
    hkv, D = k_cache.shape[1], k_cache.shape[2]
    kp = np.zeros((total, page_size, hkv, D), np.uint16)
    vp = np.zeros_like(kp)
    bt = np.full((R, maxp), -1, np.int32)
    k = 0
    for r in range(R):
        ids = perm[k:k + npg[r] + spare]
        k += npg[r] + spare
        bt[r, :len(ids)] = ids
        n = int(npg[r])
        if n:
            pad = n * page_size
            src = np.zeros((pad, hkv, D), np.uint16)
            src[:P[r]] = k_cache[kv_offsets[r]:kv_offsets[r + 1]]
            kp[ids[:n]] = src.reshape(n, page_size, hkv, D)
            src[:P[r]] = v_cache[kv_offsets[r]:kv_offsets[r + 1]]
            vp[ids[:n]] = src.reshape(n, page_size, hkv, D)
    return kp, vp, bt, P.astype(np.int32)


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def run_paged(b, m, kp, vp, bt, plen, page_size):
    import torch
    import paper_2604_09603_amd as pkg
    from paper_2604_09603_amd.step import _aligned_workspace
    cfg = b["cfg"]
    cap = cfg.R + cfg.budget
    i16 = lambda a: _dev(np.asarray(a, np.uint16).view(np.int16))
    out = torch.full((cap, cfg.hq, 128), float("nan"), dtype=torch.float32, device="cuda:0")
    lse = torch.full((cap, cfg.hq), float("nan"), dtype=torch.float32, device="cuda:0")
    status = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    ws = _aligned_workspace(pkg.tree_verify_attn_workspace_size(cfg.R, cap, cfg.hq, cfg.hkv),
                            "cuda:0")
    pkg.echo_tree_verify_attn_paged(i16(b["q"]), i16(b["k_new"]), i16(b["v_new"]), i16(kp),
                                    i16(vp), page_size, _dev(bt), _dev(plen),
                                    _dev(m["q_offsets"].astype(np.int32)),
                                    _dev(m["tree_mask"].view(np.int32)), cfg.mask_words, cfg.R,
                                    cap, cfg.hq, cfg.hkv, 128, float(b["sm_scale"]), out, lse, ws,
                                    status=status)
    torch.cuda.synchronize()
    return out.cpu().numpy(), lse.cpu().numpy(), int(status.item())


@pytest.mark.parametrize("name,page_size", [("tiny", 32), ("tiny", 256), ("l8b", 64),
                                            ("l70b", 128), ("q235b", 64), ("long", 256)])
def test_paged_attention_matches_contiguous(name, page_size):
    """Same result as the contiguous GPU path (bit for bit: these shapes run the same
    kernel in both, over the same tiles in the same order) and within tolerance of the
    oracle."""
    b = synth.make_batch(name, 0)
    ref = gc.oracle_front(b)
    m = ref["mask"]
    rng = np.random.default_rng(page_size)
    _log(f"[serve] paged {name} page_size={page_size}: building pages")
    kp, vp, bt, plen = to_pages(b["k_cache"], b["v_cache"], b["kv_offsets"], page_size, rng)
    _log(f"[serve] paged {name}: gpu")
    out, lse, status = run_paged(b, m, kp, vp, bt, plen, page_size)
    assert status == 0
    st, res = gc.run_gpu(b, ref["target"])
    nq = m["num_slots"]
    assert np.array_equal(out[:nq].view(np.uint32), res["out"][:nq].view(np.uint32))
    assert np.array_equal(lse[:nq].view(np.uint32), res["lse"][:nq].view(np.uint32))
    assert np.all(np.isnan(out[nq:]))
    rows = list(range(nq)) if name == "tiny" else gc.sample_rows(m["q_offsets"], rng)
    cfg = b["cfg"]
    ro, rl, _ = oracle.tree_verify_attn_paged(b["q"], b["k_new"], b["v_new"], kp, vp, bt, plen,
                                              page_size, m["q_offsets"], m["tree_mask"], cfg.hq,
                                              cfg.hkv, b["sm_scale"], rows=rows)
    gc.compare_attn(out, lse, ro, rl, rows)


# (Hq, Hkv, slots, keys as a function of the workgroups, same): few rows over one or
# three KV heads, where the contiguous call's kv_rows decide which main kernel runs and
# the paged call keeps the ordinary one; 128 rows; and more, where both take the
# shared-ring kernel.  same: both calls run the same kernel
POOL_CASES = [
    (8, 1, 3, lambda nb: 900, True), (8, 1, 3, lambda nb: 32 * 32 * nb - 1, True),
    (8, 1, 3, lambda nb: 64 * 32 * nb, False), (6, 3, 3, lambda nb: 32 * 32 * nb, False),
    (64, 4, 8, lambda nb: 9000, False), (64, 4, 9, lambda nb: 9000, True),
    (16, 4, 3, lambda nb: 9000, True)]


@pytest.mark.parametrize("case", range(len(POOL_CASES)))
def test_paged_attention_pool_size_does_not_matter(case):
    """The pool and the table's rows may be any times larger than the prefixes without a
    change of the result, with small tables (whose ids the plan checks) and large ones.
    The contiguous call gives the same bits where it runs the same kernel, and the same
    result to the bf16 weights' precision elsewhere."""
    import torch
    import paper_2604_09603_amd as pkg
    from paper_2604_09603_amd.step import _aligned_workspace
    hq, hkv, slots, total, same = POOL_CASES[case]
    T = total(torch.cuda.get_device_properties(0).multi_processor_count)
    R, S = 5, 256
    rng = np.random.default_rng(case)
    cuts = np.sort(rng.integers(0, T + 1, R - 1)) if T < 1 << 16 else np.arange(1, R) * (T // R) + 7
    kvo = np.concatenate([[0], cuts, [T]]).astype(np.int64)
    P = np.diff(kvo)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(case)
    normal = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda:0").normal_(  # noqa: E731
        generator=gen).view(torch.int16)
    nq = R * slots
    q, kn, vn = normal(nq, hq, 128), normal(nq, hkv, 128), normal(nq, hkv, 128)
    kc, vc = normal(T, hkv, 128), normal(T, hkv, 128)
    mask = _dev(np.tile((2 << np.arange(slots)) - 1, R).astype(np.int32))
    qo = _dev(np.arange(R + 1, dtype=np.int32) * slots)
    ws = _aligned_workspace(pkg.tree_verify_attn_workspace_size(R, nq, hq, hkv), "cuda:0")
    new = lambda *s: torch.full(s, float("nan"), device="cuda:0")  # noqa: E731
    ref, ref_lse = new(nq, hq, 128), new(nq, hq)
    _log(f"[serve] pool size: {hq}/{hkv} heads, {T} keys")
    pkg.echo_tree_verify_attn(q, kn, vn, kc, vc, _dev(kvo), T, qo, mask, 1, R, nq, hq, hkv, 128,
                              0.088, ref, ref_lse, ws)
    assert not torch.isnan(ref).any()
    npg = (P + S - 1) // S
    got = []
    for spare, row in ((0, int(npg.max())), (3 * int(npg.sum()) + 40 * hkv + 4000, 4 * int(npg.max()) + 900)):
        ids = rng.permutation(int(npg.sum()) + spare)[:int(npg.sum())]
        bt = np.full((R, row), -1, np.int32)
        dest = np.empty(T, np.int64)
        for r in range(R):
            mine = ids[npg[:r].sum():npg[:r + 1].sum()]
            bt[r, :npg[r]] = mine
            at = np.arange(P[r])
            dest[kvo[r]:kvo[r + 1]] = mine[at // S] * S + at % S
        pages = []
        for c in (kc, vc):
            t = torch.zeros(((len(ids) + spare) * S, hkv, 128), dtype=torch.int16, device="cuda:0")
            t[_dev(dest)] = c
            pages.append(t.view(-1, S, hkv, 128))
        out, lse = new(nq, hq, 128), new(nq, hq)
        status = torch.zeros(1, dtype=torch.int32, device="cuda:0")
        pkg.echo_tree_verify_attn_paged(q, kn, vn, *pages, S, _dev(bt), _dev(P.astype(np.int32)), qo,
                                        mask, 1, R, nq, hq, hkv, 128, 0.088, out, lse, ws,
                                        status=status)
        assert int(status.item()) == 0
        got.append((out.view(torch.int32), lse.view(torch.int32)))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    if same:
        assert torch.equal(got[0][0], ref.view(torch.int32))
        assert torch.equal(got[0][1], ref_lse.view(torch.int32))
    else:
        # two roundings of the weights to bf16: see compare_attn's bounds
        scale = ref.abs().amax(-1, keepdim=True)
        assert ((got[0][0].view(torch.float32) - ref).abs() <= 2 * gc.RTOL_ROW * scale).all()
        assert (got[0][1].view(torch.float32) - ref_lse).abs().max() <= 2 * gc.LSE_ATOL


def test_paged_attention_missing_page_skips_the_request():
    b = synth.make_batch("tiny", 3)
    ref = gc.oracle_front(b)
    m = ref["mask"]
    kp, vp, bt, plen = to_pages(b["k_cache"], b["v_cache"], b["kv_offsets"], 64,
                                np.random.default_rng(1))
    bt[2, 1] = -1                                    # request 2 loses its second page
    out, lse, status = run_paged(b, m, kp, vp, bt, plen, 64)
    assert status & oracle.status.BAD_OFFSETS
    q0, q1 = int(m["q_offsets"][2]), int(m["q_offsets"][3])
    assert np.all(np.isnan(out[q0:q1]))
    cfg = b["cfg"]
    rows = [s for s in range(m["num_slots"]) if not q0 <= s < q1]
    ro, rl, _ = oracle.tree_verify_attn_paged(b["q"], b["k_new"], b["v_new"], kp, vp, bt, plen,
                                              64, m["q_offsets"], m["tree_mask"], cfg.hq, cfg.hkv,
                                              b["sm_scale"], rows=rows)
    gc.compare_attn(out, lse, ro, rl, rows)


@pytest.mark.parametrize("R,max_pages", [(1, 1), (1, 4096), (1, 4097), (3, 1365), (3, 1366),
                                         (256, 16), (256, 17), (257, 15)])
def test_paged_attention_page_check_sizes(R, max_pages):
    """Around the size up to which the plan checks the page ids itself: a bad id in the
    table's very last entry, a length past the table row, ids past the prefix that don't
    count."""
    import types
    S = 32
    rng = np.random.default_rng(R * 10007 + max_pages)
    kp, vp = (synth.f32_to_bf16_bits(rng.standard_normal((40, S, 1, 128)).astype(np.float32))
              for _ in range(2))
    q, kn, vn = (synth.f32_to_bf16_bits(rng.standard_normal((R, 1, 128)).astype(np.float32))
                 for _ in range(3))
    cfg = types.SimpleNamespace(R=R, budget=0, hq=1, hkv=1, mask_words=1)
    b = dict(cfg=cfg, q=q, k_new=kn, v_new=vn, sm_scale=128 ** -0.5)
    m = dict(q_offsets=np.arange(R + 1, dtype=np.int32),
             tree_mask=np.ones((R, 1), np.uint32))
    plen = rng.integers(0, min(max_pages, 6) * S + 1, R).astype(np.int32)
    plen[-1] = max_pages * S - 5
    bt = rng.integers(0, 40, (R, max_pages)).astype(np.int32)
    for r in range(R):
        bt[r, (plen[r] + S - 1) // S:] = -1 if r % 2 else 40
    for spoil in ("none", "last id", "length"):
        t, n = bt.copy(), plen.copy()
        skipped = -1
        if spoil == "last id":
            skipped = R - 1
            t[skipped, -1] = 40
        elif spoil == "length":
            skipped = R // 2
            n[skipped] = max_pages * S + 1
        _log(f"[serve] page check R={R} max_pages={max_pages} spoil={spoil}")
        out, lse, status = run_paged(b, m, kp, vp, t, n, S)
        assert status == (0 if skipped < 0 else oracle.status.BAD_OFFSETS)
        rows = [s for s in (range(R) if R <= 3 else (0, 1, R // 2, R - 2, R - 1)) if s != skipped]
        assert skipped < 0 or np.all(np.isnan(out[skipped]))
        assert not np.any(np.isnan(np.delete(out, [skipped], 0) if skipped >= 0 else out))
        if not rows:
            continue
        if skipped >= 0:
            n[skipped] = 0  # (the oracle is given the valid requests)
        ro, rl, _ = oracle.tree_verify_attn_paged(q, kn, vn, kp, vp, t, n, S, m["q_offsets"],
                                                  m["tree_mask"], 1, 1, b["sm_scale"], rows=rows)
        gc.compare_attn(out, lse, ro, rl, rows)


def _accept_logits_case(b, m, vocab, rng, ties=True, nan_rows=0):
    import torch
    import paper_2604_09603_amd as pkg
    cfg = b["cfg"]
    cap = cfg.R + cfg.budget
    nq = m["num_slots"]
    if ties:   # few distinct values: ties are everywhere
        vals = torch.randint(-6, 6, (cap, vocab), dtype=torch.int32, device="cuda:0")
        logits = (vals.float() * 0.5).to(torch.bfloat16)
    else:
        logits = (torch.randn(cap, vocab, device="cuda:0") * 3).to(torch.bfloat16)
    for i in range(nan_rows):
        logits[i * 3, ::7] = float("nan")
        if i == 0:
            logits[0, :] = float("nan")
    lg = logits.view(torch.int16)
    d = lambda a: _dev(np.asarray(a, np.int32))
    tgt = torch.full((cap,), -7, dtype=torch.int32, device="cuda:0")
    al = torch.zeros(cfg.R, dtype=torch.int32, device="cuda:0")
    aslots = torch.zeros((cfg.R, 16), dtype=torch.int32, device="cuda:0")
    bonus = torch.zeros(cfg.R, dtype=torch.int32, device="cuda:0")
    status = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    pkg.echo_accept_logits(d(m["q_offsets"]), d(m["slot_parent"]), d(m["slot_token"]), lg, cfg.R,
                           cap, 16, tgt, al, aslots, bonus, status=status)
    torch.cuda.synchronize()
    host_logits = lg.cpu().numpy().view(np.uint16)
    want = oracle.accept_from_logits(m["q_offsets"], m["slot_parent"], m["slot_token"],
                                     host_logits, 16)
    t = tgt.cpu().numpy()
    assert np.array_equal(t[:nq], want["target_token"]), "argmax differs"
    assert np.all(t[nq:] == -7)
    assert np.array_equal(al.cpu().numpy(), want["accept_len"])
    assert np.array_equal(aslots.cpu().numpy(), want["accept_slots"])
    assert np.array_equal(bonus.cpu().numpy(), want["bonus_token"])
    assert int(status.item()) == want["status"]


@pytest.mark.parametrize("name,vocab,ties", [("tiny", 32, True), ("tiny", 1001, True),
                                             ("l8b", 128256, False), ("q235b", 151936, True),
                                             ("q235b", 151937, False)])
def test_accept_from_logits(name, vocab, ties):
    b = synth.make_batch(name, 1)
    ref = gc.oracle_front(b)
    _log(f"[serve] accept_logits {name} V={vocab} ties={ties}")
    _accept_logits_case(b, ref["mask"], vocab, np.random.default_rng(0), ties=ties,
                        nan_rows=2 if name == "tiny" else 0)


@pytest.mark.parametrize("vocab", [1, 7, 8, 9, 40959, 81920 + 8, 49153])
@pytest.mark.parametrize("rows", [5, 300])
def test_target_argmax_edges(vocab, rows):
    """Row lengths on both sides of the 16-byte blocks (odd ones misalign the rows)
    and of the batches of 10 x 512 and 5 x 1024 blocks, few rows and more than the
    GPU has CUs; in the first rows what integer order does not decide: NaN of both
    signs, a largest value of zero with both signs, only -inf, -inf and NaN, only
    NaN.  Against the oracle, exactly."""
    import torch
    import paper_2604_09603_amd as pkg
    rng = np.random.default_rng(vocab + rows)
    vals = rng.integers(-40, 3, (rows, vocab)).astype(np.float32) / 4
    bits = synth.f32_to_bf16_bits(vals).reshape(rows, vocab).copy()
    neg = (bits >> 15) & 1
    bits[0] = np.where(rng.random(vocab) < 0.3, 0x7FC0 | (neg[0] << 15), bits[0])
    bits[1] = np.where(vals[1] >= 0, np.where(rng.random(vocab) < 0.5, 0x8000, 0), bits[1])
    bits[2] = 0xFF80
    bits[3] = np.where(rng.random(vocab) < 0.5, 0xFF80, 0x7F81)
    bits[4] = np.where(rng.random(vocab) < 0.5, 0xFFC1, 0x7FC0)
    i32 = lambda *s: torch.zeros(s, dtype=torch.int32, device="cuda:0")
    target = i32(rows)
    qo = np.arange(rows + 1, dtype=np.int32)
    _log(f"[serve] argmax V={vocab} rows={rows}")
    pkg.echo_accept_logits(_dev(qo), _dev(np.full(rows, -1, np.int32)), i32(rows),
                           _dev(bits.view(np.int16)), rows, rows, 16, target, i32(rows),
                           i32(rows, 16), i32(rows))
    torch.cuda.synchronize()
    want = oracle.accept_from_logits(qo, np.full(rows, -1, np.int32), np.zeros(rows, np.int32),
                                     bits, 16)
    assert np.array_equal(target.cpu().numpy(), want["target_token"])


@pytest.mark.parametrize("vocab", [9, 1000, 8200, 40959, 40969, 90001])
@pytest.mark.parametrize("rows", [7, 300])
def test_target_argmax_negative_rows(vocab, rows):
    """Rows without a positive logit, whose order is by the bit patterns' other end: ties,
    NaN of both signs among them, a largest logit of -0 alone, -inf beside NaN; and a
    maximum in the last block and in the last element.  Against the oracle, exactly."""
    import torch
    import paper_2604_09603_amd as pkg
    rng = np.random.default_rng(vocab + 3 * rows)
    vals = -(rng.integers(1, 200, (rows, vocab)).astype(np.float32)) / 4
    bits = synth.f32_to_bf16_bits(vals).reshape(rows, vocab).copy()
    bits[1] = np.where(rng.random(vocab) < 0.2, 0x7FC0, np.where(rng.random(vocab) < 0.2, 0xFFC0, bits[1]))
    bits[2, rng.integers(0, vocab, 3)] = 0x8000
    bits[3] = np.where(rng.random(vocab) < 0.5, 0xFF80, np.where(rng.random(vocab) < 0.5, 0xFFFF, 0x7F81))
    bits[4, vocab - 1] = 0x0001
    bits[5, (vocab - 1) // 8 * 8 - (8 if vocab > 8 else 0)] = 0x3F80
    bits[6] = 0x7F80 if vocab == 9 else 0x8000
    i32 = lambda *s: torch.zeros(s, dtype=torch.int32, device="cuda:0")
    target = i32(rows)
    qo, par = np.arange(rows + 1, dtype=np.int32), np.full(rows, -1, np.int32)
    _log(f"[serve] argmax of negative logits V={vocab} rows={rows}")
    pkg.echo_accept_logits(_dev(qo), _dev(par), i32(rows), _dev(bits.view(np.int16)), rows, rows,
                           16, target, i32(rows), i32(rows, 16), i32(rows))
    torch.cuda.synchronize()
    want = oracle.accept_from_logits(qo, par, np.zeros(rows, np.int32), bits, 16)
    assert np.array_equal(target.cpu().numpy(), want["target_token"])


def test_commit_kv_matches_oracle():
    import torch
    import paper_2604_09603_amd as pkg
    b = synth.make_batch("l8b", 2)
    ref = gc.oracle_front(b)
    m, a = ref["mask"], ref["accept"]
    cfg = b["cfg"]
    cap = cfg.R + cfg.budget
    rng = np.random.default_rng(4)
    page_size = 16
    kp, vp, bt, plen = to_pages(b["k_cache"], b["v_cache"], b["kv_offsets"], page_size, rng,
                                spare=3)
    bt[5, :] = -1                                     # request 5 has no pages: refused
    d32 = lambda x: _dev(np.asarray(x, np.int32))
    i16 = lambda x: _dev(np.asarray(x, np.uint16).view(np.int16))
    kpd, vpd, pld = i16(kp), i16(vp), d32(plen)
    status = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    pkg.echo_commit_kv(d32(m["q_offsets"]), d32(a["accept_len"]), d32(a["accept_slots"]), 16,
                       i16(b["k_new"]), i16(b["v_new"]), cfg.R, cap, cfg.hkv, kpd, vpd,
                       page_size, d32(bt), pld, status=status)
    torch.cuda.synchronize()
    kp2, vp2, P2, s = oracle.commit_kv(m["q_offsets"], a["accept_len"], a["accept_slots"],
                                       b["k_new"], b["v_new"], kp, vp, bt, plen, page_size)
    assert np.array_equal(pld.cpu().numpy(), P2)
    assert np.array_equal(kpd.cpu().numpy().view(np.uint16), kp2)
    assert np.array_equal(vpd.cpu().numpy().view(np.uint16), vp2)
    assert int(status.item()) == s == oracle.status.BAD_OFFSETS


def test_serving_step_with_paged_cache():
    """gate -> mask -> paged attention -> accept from logits -> commit, then a
    second verification over the grown cache, on the tiny preset."""
    import torch
    import paper_2604_09603_amd as pkg
    from paper_2604_09603_amd.step import VerifyStep, _aligned_workspace
    b = synth.make_batch("tiny", 4)
    cfg = b["cfg"]
    cap = cfg.R + cfg.budget
    rng = np.random.default_rng(6)
    page_size = 32
    kp, vp, bt, plen = to_pages(b["k_cache"], b["v_cache"], b["kv_offsets"], page_size, rng,
                                spare=2)
    st = VerifyStep(b)
    st.gate()
    st.mask()
    res = st.fetch()
    ref = gc.oracle_front(b)
    m = ref["mask"]
    out, lse, status = run_paged(b, m, kp, vp, bt, plen, page_size)
    assert status == 0
    logits = (torch.randn(cap, 32, device="cuda:0") * 2).to(torch.bfloat16).view(torch.int16)
    d32 = lambda x: _dev(np.asarray(x, np.int32))
    i16 = lambda x: _dev(np.asarray(x, np.uint16).view(np.int16))
    tgt = torch.zeros(cap, dtype=torch.int32, device="cuda:0")
    pkg.echo_accept_logits(st.q_offsets, st.slot_parent, st.slot_token, logits, cfg.R, cap, 16,
                           tgt, st.accept_len, st.accept_slots, st.bonus_token, status=st.status)
    kpd, vpd, pld, btd = i16(kp), i16(vp), d32(plen), d32(bt)
    pkg.echo_commit_kv(st.q_offsets, st.accept_len, st.accept_slots, 16, st.k_new, st.v_new,
                       cfg.R, cap, cfg.hkv, kpd, vpd, page_size, btd, pld, status=st.status)
    torch.cuda.synchronize()
    hl = logits.cpu().numpy().view(np.uint16)
    acc = oracle.accept_from_logits(m["q_offsets"], m["slot_parent"], m["slot_token"], hl, 16)
    kp2, vp2, P2, s = oracle.commit_kv(m["q_offsets"], acc["accept_len"], acc["accept_slots"],
                                       b["k_new"], b["v_new"], kp, vp, bt, plen, page_size)
    assert s == 0 and int(st.status.item()) == 0
    assert np.array_equal(st.accept_len.cpu().numpy(), acc["accept_len"])
    assert np.array_equal(pld.cpu().numpy(), P2)
    assert np.array_equal(kpd.cpu().numpy().view(np.uint16), kp2)
    # next step: every request verifies one new root over the grown prefix
    q1 = np.asarray(b["q"][:cfg.R])
    qo1 = np.arange(cfg.R + 1, dtype=np.int32)
    mask1 = np.zeros((cap, cfg.mask_words), np.uint32)
    mask1[:cfg.R, 0] = 1
    b2 = dict(b, q=np.concatenate([q1, np.zeros((cfg.budget,) + q1.shape[1:], np.uint16)]))
    out2, lse2, st2 = run_paged(b2, dict(q_offsets=qo1, tree_mask=mask1), kp2, vp2, bt, P2,
                                page_size)
    assert st2 == 0
    ro, rl, _ = oracle.tree_verify_attn_paged(b2["q"], b["k_new"], b["v_new"], kp2, vp2, bt, P2,
                                              page_size, qo1, mask1, cfg.hq, cfg.hkv,
                                              b["sm_scale"])
    gc.compare_attn(out2, lse2, ro, rl, range(cfg.R))


@pytest.mark.parametrize("hq,hkv,page_size", [(8, 1, 32), (15, 5, 64), (56, 7, 32), (96, 3, 64)])
def test_paged_attention_head_layouts(hq, hkv, page_size):
    """The paged path over unusual head layouts (one KV head, KV-head counts
    that are not powers of two, GQA up to 32, several row passes per head):
    bit for bit the contiguous GPU path, and every row against the oracle."""
    from tests.test_gpu_edges import make_micro_batch, _front_ref
    rng = np.random.default_rng(hq * 1000 + hkv * 10 + page_size)
    pool = synth.micro_pool(rng, int(rng.integers(3, 24)), 30, p_neg_inf=0.05)
    N = int(pool["cand_offsets"][-1])
    b = make_micro_batch(pool, max(1, N * 3 // 4), hq=hq, hkv=hkv, p_range=(0, 300),
                         seed=hq + hkv + page_size)
    ref = _front_ref(b)
    m = ref["mask"]
    _log(f"[serve] paged layouts hq={hq} hkv={hkv} page_size={page_size}")
    kp, vp, bt, plen = to_pages(b["k_cache"], b["v_cache"], b["kv_offsets"], page_size, rng)
    out, lse, status = run_paged(b, m, kp, vp, bt, plen, page_size)
    assert status == 0
    st, res = gc.run_gpu(b, ref["target"])
    nq = m["num_slots"]
    assert np.array_equal(out[:nq].view(np.uint32), res["out"][:nq].view(np.uint32))
    assert np.array_equal(lse[:nq].view(np.uint32), res["lse"][:nq].view(np.uint32))
    cfg = b["cfg"]
    rows = list(range(nq))
    ro, rl, _ = oracle.tree_verify_attn_paged(b["q"], b["k_new"], b["v_new"], kp, vp, bt, plen,
                                              page_size, m["q_offsets"], m["tree_mask"], cfg.hq,
                                              cfg.hkv, b["sm_scale"], rows=rows)
    gc.compare_attn(out, lse, ro, rl, rows)
