"""Chunked prefill (tool observations appended as multi-token chunks) on the
GPU against the CPU reference: whole layers with mixed decode and prefill
sequences, the attention call alone under sink stress and page permutation,
and the full-size mixed step (192 decode sequences plus 64 chunks of
256-4096 tokens) on sampled sequences.

Sequences adding 16 or more tokens take the prefill kernel (blocks of 32
tokens for 8 query heads per KV head, 64 for 4); shorter additions take the
split-K decode path, so the cases below cover both sides of that boundary,
ragged last blocks, empty contexts and windows shorter than the chunk.
"""
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2608_22167_amd import mcpu, workload as W
from tests import parity as PT
from tests.test_gpu_parity import compare_layer, reference, run_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    torch.cuda.set_device(0)
    yield
    torch.cuda.empty_cache()


def test_prefill_tiny_f32_layer():
    shape = W.TINY  # 4 query heads per KV head: 64-token blocks
    wl = W.custom(shape, [0, 10, 100, 250, 3], [20, 70, 1, 130, 15], 1101, sink_std=1.0)
    gpu, step = run_layer(wl)
    compare_layer(wl, gpu, step)


@pytest.mark.parametrize("hq,hkv", [(16, 1), (4, 2)])
def test_prefill_head_groupings_without_prefill_kernel(hq, hkv):
    """16 and 2 query heads per KV head have no prefill-kernel instance: their
    chunks go to split-K attention, with the same results."""
    shape = replace(W.TINY, n_q_heads=hq, n_kv_heads=hkv)
    wl = W.custom(shape, [0, 10, 100, 3], [20, 70, 1, 33], 1105 + hq, sink_std=1.0)
    gpu, step = run_layer(wl)
    compare_layer(wl, gpu, step)


@pytest.mark.parametrize("window", [0, 128])
def test_prefill_bf16_layer(window):
    shape = replace(W.GPT_OSS_20B, window=window)
    wl = W.custom(shape, [0, 3, 200, 1500, 40], [40, 17, 1, 300, 15], 1102 + window, sink_std=0.5)
    gpu, step = run_layer(wl)
    compare_layer(wl, gpu, step)


def _attention(wl, sinks, pool_k, pool_v, page_table, q_scale=1.0):
    s = wl.shape
    T = wl.n_tokens
    q = W.synth_normal(wl.seed, 901, (T, s.n_q_heads, s.head_dim), std=q_scale, dtype=s.torch_dtype)
    pool = mcpu.KVPool(s, pool_k.cuda(), pool_v.cuda())
    o = torch.empty((T, s.n_q_heads * s.head_dim), dtype=s.torch_dtype, device="cuda")
    ws = mcpu.workspace(mcpu.paged_attention_workspace_size(s, wl.batch, T))
    mcpu.paged_attention(s, sinks.cuda(), pool, torch.from_numpy(page_table).cuda(),
                         torch.from_numpy(wl.seq_lens).cuda(), torch.from_numpy(wl.cu_q).cuda(),
                         wl.seq_lens, wl.cu_q, q.cuda(), o, ws)
    torch.cuda.synchronize()
    assert mcpu.mcpu_check_device_errors(ws) == 0
    return q, o.cpu()


@pytest.mark.parametrize("window", [0, 128])
def test_prefill_attention_sink_stress_and_page_permutation(window):
    """Sinks far above and far below the scores, and the same step with the
    pool's pages renumbered: identical bits."""
    shape = replace(W.GPT_OSS_20B, window=window)
    wl = W.custom(shape, [0, 700, 31, 16], [64, 100, 33, 1], 1111 + window, weights=False)
    sinks = torch.from_numpy(np.tile([12.0, -12.0, 0.0, 3.0], shape.n_q_heads // 4).astype(np.float32))
    q, o = _attention(wl, sinks, wl.k_pool, wl.v_pool, wl.page_table)
    tok_seq = np.repeat(np.arange(wl.batch), wl.q_lens)
    tok_pos = np.concatenate([wl.seq_lens[b] + np.arange(wl.q_lens[b]) for b in range(wl.batch)])
    ref = O.attention(shape, tok_seq, tok_pos, q, wl.k_pool, wl.v_pool, wl.page_table, sinks)
    PT.check("prefill attention", o.float().numpy().reshape(ref.shape), ref, shape.dtype)
    perm = np.random.default_rng(7).permutation(wl.n_pages).astype(np.int32)
    inv = np.argsort(perm).astype(np.int32)
    k2 = torch.empty_like(wl.k_pool)
    v2 = torch.empty_like(wl.v_pool)
    k2[torch.from_numpy(inv).long()] = wl.k_pool
    v2[torch.from_numpy(inv).long()] = wl.v_pool
    pt2 = np.where(wl.page_table >= 0, inv[np.maximum(wl.page_table, 0)], -1).astype(np.int32)
    _, o2 = _attention(wl, sinks, k2, v2, pt2)
    assert torch.equal(o.view(torch.int16), o2.view(torch.int16))


@pytest.mark.parametrize("window", [0, 128])
def test_prefill_attention_large_scores_and_extreme_sinks(window):
    """Queries scaled x 50 (scores up to about 200, so the lazy rescale of the
    running maximum is taken on most steps) with sinks of +30 and -30: the
    max-subtracted softmax stays finite and matches the reference."""
    shape = replace(W.GPT_OSS_20B, window=window)
    wl = W.custom(shape, [0, 900, 47, 16], [96, 130, 40, 1], 1113 + window, weights=False)
    sinks = torch.from_numpy(np.tile([30.0, -30.0, 0.5, 4.0], shape.n_q_heads // 4).astype(np.float32))
    q, o = _attention(wl, sinks, wl.k_pool, wl.v_pool, wl.page_table, q_scale=50.0)
    tok_seq = np.repeat(np.arange(wl.batch), wl.q_lens)
    tok_pos = np.concatenate([wl.seq_lens[b] + np.arange(wl.q_lens[b]) for b in range(wl.batch)])
    ref = O.attention(shape, tok_seq, tok_pos, q, wl.k_pool, wl.v_pool, wl.page_table, sinks)
    got = o.float().numpy().reshape(ref.shape)
    assert np.isfinite(got).all()
    PT.check("prefill attention (q x 50, sinks +-30)", got, ref, shape.dtype)
    assert np.abs(got[:, 1::4]).max() > 0.1   # the -30 sink heads: peaked, not averaged away


def _run_layer_rows(wl, rows):
    """decode_layer on the whole step; only the given token rows come back."""
    step = mcpu.DeviceStep(wl)
    s = wl.shape
    T = wl.n_tokens
    taps_t = dict(q=torch.empty((T, s.n_q_heads, s.head_dim), dtype=s.torch_dtype, device="cuda"),
                  o=torch.empty((T, s.attn_dim), dtype=s.torch_dtype, device="cuda"),
                  h1=torch.empty((T, s.hidden), dtype=torch.float32, device="cuda"))
    step.run(mcpu.Taps(q=taps_t["q"].data_ptr(), o=taps_t["o"].data_ptr(), h1=taps_t["h1"].data_ptr()))
    torch.cuda.synchronize()
    assert step.device_errors() == 0
    r = torch.from_numpy(np.asarray(rows, np.int64)).cuda()
    pick = lambda t: t.index_select(0, r).float().cpu().numpy().astype(np.float64)
    out = dict(out=pick(step.x_out), idx=step.topk_idx.index_select(0, r).cpu().numpy(), w=pick(step.topk_w),
               q=pick(taps_t["q"]), o=pick(taps_t["o"]), h1=pick(taps_t["h1"]))
    finite = bool(torch.isfinite(step.x_out).all())
    wsum = step.topk_w.sum(1)
    wsum_ok = bool(((wsum - 1).abs() <= 1e-5).all())
    return out, finite, wsum_ok


def test_mixed_step_full_size_sampled():
    """The 192 + 64 sequence mixed step at full size (151k tokens), compared on
    two decode sequences and the prefill sequence with the shortest chunk."""
    wl = W.mixed_prefill()
    dec = np.nonzero(wl.q_lens == 1)[0]
    pre = np.nonzero(wl.q_lens > 1)[0]
    seqs = sorted({int(dec[np.argmax(wl.seq_lens[dec])]), int(dec[0]), int(pre[np.argmin(wl.q_lens[pre])])})
    sub, rows = W.restrict(wl, seqs)
    g, finite, wsum_ok = _run_layer_rows(wl, rows)
    assert finite and wsum_ok
    ref, _ = reference(sub, g)
    compare_layer(sub, g, None, ref)


def test_mixed_step_full_size_longest_chunk_sampled():
    """The full-size mixed step on the prefill sequence with the longest
    context among those adding at least 2048 tokens: every chunk token is
    appended by the reference, and a seeded subset of its rows (first, last
    and eight others) goes through attention, the output projection and the
    MoE, so the chunk's ring of pages is compared at full depth."""
    wl = W.mixed_prefill()
    pre = np.nonzero(wl.q_lens >= 2048)[0]
    b = int(pre[np.argmax(wl.seq_lens[pre])])
    sub, rows = W.restrict(wl, [b])
    n = int(wl.q_lens[b])
    rng = np.random.default_rng(1114)
    local = np.unique(np.concatenate([[0, n - 1], rng.choice(n, 8, replace=False)])).astype(np.int32)
    g, finite, wsum_ok = _run_layer_rows(wl, np.asarray(rows)[local])
    assert finite and wsum_ok
    print(f"  sequence {b}: {int(wl.seq_lens[b])} cached + {n} new tokens, rows {local.tolist()}")
    ref = O.decode_layer(sub, rows=local)
    tie = PT.check_router(g["idx"], ref["idx"], ref["logits"], sub.shape.top_k)
    if tie.any():
        force = np.zeros((sub.n_tokens, sub.shape.top_k), np.int32)
        force[local] = ref["idx"]
        force[local[tie]] = g["idx"][tie]
        ref = O.decode_layer(sub, rows=local, force_idx=force)
    compare_layer(sub, g, None, ref)


@pytest.mark.parametrize("scale", [1.0, 40.0, -40.0])
@pytest.mark.parametrize("window", [0, 128])
@pytest.mark.parametrize("hq,hkv", [(16, 2), (8, 2)])
def test_prefill_score_range(hq, hkv, window, scale):
    """Chunks whose scores climb (or fall) along the context, at scale 40 by
    thousands of powers of two: the running maximum starts at a column's first
    visible key, is raised when weights leave the range, and earlier weights
    vanish. Chunks shorter than a block, past one, and behind 0, 13, 500 and
    2000 cached keys (more than one block of page ids); with and without sinks.
    Scores are large, so the softmax is nearly one-hot: bf16 storage of q, k, v,
    the weights and o bounds the difference."""
    s = replace(W.GPT_OSS_20B, hidden=256, n_q_heads=hq, n_kv_heads=hkv, window=window)
    wl = W.custom(s, [0, 13, 500, 2000], [17, 70, 33, 40], 1190, weights=False)
    rng = np.random.default_rng(7)
    T = wl.n_tokens
    q = torch.from_numpy(rng.standard_normal((T, hq, 64)).astype(np.float32))
    # a common direction in q and k whose weight grows with the position
    d = torch.from_numpy(rng.standard_normal(64).astype(np.float32))
    q = (q + d * scale).to(torch.bfloat16)
    k = wl.k_pool.float()
    for b in range(wl.batch):
        for lp, page in enumerate(wl.page_table[b]):
            if page >= 0:  # [hkv, 16, 64] in page order; dims run in blocks of 8: [8][16][8]
                k[page] += (lp / 20.0) * d.view(8, 1, 8).expand(8, 16, 8).reshape(1, 16, 64)
    k = k.to(torch.bfloat16)
    for sinks in (None, torch.linspace(-3, 3, hq)):
        o = torch.empty((T, hq * 64), dtype=torch.bfloat16, device="cuda")
        kd, vd = k.cuda(), wl.v_pool.cuda()
        ws = mcpu.workspace(mcpu.paged_attention_workspace_size(s, wl.batch, T))
        mcpu.paged_attention(s, None if sinks is None else sinks.cuda(), mcpu.KVPool(s, kd, vd),
                             torch.from_numpy(wl.page_table).cuda(), torch.from_numpy(wl.seq_lens).cuda(),
                             torch.from_numpy(wl.cu_q).cuda(), wl.seq_lens, wl.cu_q, q.cuda(), o, ws)
        torch.cuda.synchronize()
        assert mcpu.mcpu_check_device_errors(ws) == 0
        seq = np.repeat(np.arange(wl.batch), wl.q_lens)
        pos = np.concatenate([np.arange(l, l + n) for l, n in zip(wl.seq_lens, wl.q_lens)])
        ref = O.attention(s, seq, pos, q.double().numpy(), k.float().numpy(), wl.v_pool.float().numpy(), wl.page_table,
                          None if sinks is None else sinks.numpy())
        PT.check("o", o.float().cpu().double().numpy().reshape(ref.shape), ref, "bf16")


@pytest.mark.parametrize("window", [0, 128])
def test_prefill_large_values(window):
    """Values of 2^108 behind scores that climb by about four powers of two per
    page: weights stay within 2^8 of the running maximum, so the accumulators
    stay below 2^8 x 2^111 x a few keys, in range of fp32 (weights let run to
    2^20 would leave it)."""
    s = replace(W.GPT_OSS_20B, hidden=256, n_q_heads=16, n_kv_heads=2, window=window)
    wl = W.custom(s, [0, 100, 300], [17, 40, 70], 1192, weights=False)
    rng = np.random.default_rng(8)
    T = wl.n_tokens
    d = torch.from_numpy(rng.choice([-1.0, 1.0], 64).astype(np.float32))
    q = (torch.from_numpy(rng.standard_normal((T, 16, 64)).astype(np.float32)) * 0.1 + d).to(torch.bfloat16)
    k = wl.k_pool.float() * 0.1
    for b in range(wl.batch):
        for lp, page in enumerate(wl.page_table[b]):
            if page >= 0:
                k[page] += 0.375 * lp * d.view(8, 1, 8).expand(8, 16, 8).reshape(1, 16, 64)
    k, v = k.to(torch.bfloat16), (wl.v_pool.float() * 2.0 ** 108).to(torch.bfloat16)
    o = torch.empty((T, 16 * 64), dtype=torch.bfloat16, device="cuda")
    ws = mcpu.workspace(mcpu.paged_attention_workspace_size(s, wl.batch, T))
    mcpu.paged_attention(s, None, mcpu.KVPool(s, k.cuda(), v.cuda()),
                         torch.from_numpy(wl.page_table).cuda(), torch.from_numpy(wl.seq_lens).cuda(),
                         torch.from_numpy(wl.cu_q).cuda(), wl.seq_lens, wl.cu_q, q.cuda(), o, ws)
    torch.cuda.synchronize()
    assert mcpu.mcpu_check_device_errors(ws) == 0
    seq = np.repeat(np.arange(wl.batch), wl.q_lens)
    pos = np.concatenate([np.arange(l, l + n) for l, n in zip(wl.seq_lens, wl.q_lens)])
    ref = O.attention(s, seq, pos, q.double().numpy(), k.float().numpy(), wl.v_pool.float().numpy(), wl.page_table, None)
    PT.check("o", (o.double().cpu() * 2.0 ** -108).numpy().reshape(ref.shape), ref, "bf16")


@pytest.mark.parametrize("hq,hkv", [(16, 2), (8, 2)])
def test_prefill_pools_off_16_byte_boundaries(hq, hkv):
    """Pools that start 8 bytes past a 16-byte boundary, which direct loads to
    LDS are not used on: chunks of one block, past one and behind cached keys."""
    s = replace(W.GPT_OSS_20B, hidden=256, n_q_heads=hq, n_kv_heads=hkv, window=0)
    wl = W.custom(s, [0, 13, 500], [17, 70, 40], 1193, weights=False)
    T = wl.n_tokens
    q = W.synth_normal(1193, 40, (T, hq, 64), dtype=torch.bfloat16)
    pools = []
    for p in (wl.k_pool, wl.v_pool):
        buf = torch.empty(p.numel() + 4, dtype=p.dtype, device="cuda")
        buf[4:].copy_(p.view(-1))
        pools.append(buf[4:].view(p.shape))
        assert pools[-1].data_ptr() % 16 == 8
    o = torch.empty((T, hq * 64), dtype=torch.bfloat16, device="cuda")
    ws = mcpu.workspace(mcpu.paged_attention_workspace_size(s, wl.batch, T))
    mcpu.paged_attention(s, None, mcpu.KVPool(s, *pools), torch.from_numpy(wl.page_table).cuda(),
                         torch.from_numpy(wl.seq_lens).cuda(), torch.from_numpy(wl.cu_q).cuda(), wl.seq_lens, wl.cu_q,
                         q.cuda(), o, ws)
    torch.cuda.synchronize()
    assert mcpu.mcpu_check_device_errors(ws) == 0
    seq = np.repeat(np.arange(wl.batch), wl.q_lens)
    pos = np.concatenate([np.arange(l, l + n) for l, n in zip(wl.seq_lens, wl.q_lens)])
    ref = O.attention(s, seq, pos, q.double().numpy(), wl.k_pool.float().numpy(), wl.v_pool.float().numpy(),
                      wl.page_table, None)
    PT.check("o", o.float().cpu().double().numpy().reshape(ref.shape), ref, "bf16")


@pytest.mark.parametrize("case", ["many_seqs", "many_tokens", "one_long", "wave_edges", "in_order"])
def test_plan_and_combine_edges(case):
    """Sizes at which the plan and the merge of splits change form: more
    sequences than are searched in LDS (2048), more tokens than one per thread
    (4096) and than one token per wavefront of the merge (65536 / 16 heads), one
    token with more splits than a wavefront has lanes, split counts around a
    wavefront's rows per load, and one to nine splits among enough tokens to be
    merged in order. Chunks of 1-3 tokens stay on the split path."""
    s = replace(W.GPT_OSS_20B, hidden=256, n_q_heads=16, n_kv_heads=2, window=0)
    rng = np.random.default_rng(11)
    if case == "many_seqs":
        lens, q = rng.integers(0, 40, 2100), rng.integers(1, 3, 2100)
    elif case == "many_tokens":
        lens, q = rng.integers(0, 60, 1500), rng.integers(2, 5, 1500)
    elif case == "one_long":
        lens, q = np.array([9001]), np.array([1])
    elif case == "in_order":
        lens, q = np.concatenate([rng.integers(0, 40, 500), 255 + 256 * np.arange(9)]), np.ones(509, int)
    else:
        lens, q = np.array([15, 16, 63, 64, 500, 1023, 1024, 2100, 0]), np.array([1, 1, 2, 1, 3, 1, 1, 1, 1])
    wl = W.custom(s, [int(x) for x in lens], [int(x) for x in q], 1191, weights=False)
    T = wl.n_tokens
    if case == "many_tokens":
        assert T > 4096 and T * s.n_q_heads > 65536
    qv = torch.from_numpy(rng.standard_normal((T, s.n_q_heads, 64)).astype(np.float32)).to(torch.bfloat16)
    sinks = torch.linspace(-2, 2, s.n_q_heads)
    o = torch.empty((T, s.n_q_heads * 64), dtype=torch.bfloat16, device="cuda")
    ws = mcpu.workspace(mcpu.paged_attention_workspace_size(s, wl.batch, T))
    mcpu.paged_attention(s, sinks.cuda(), mcpu.KVPool(s, wl.k_pool.cuda(), wl.v_pool.cuda()),
                         torch.from_numpy(wl.page_table).cuda(), torch.from_numpy(wl.seq_lens).cuda(),
                         torch.from_numpy(wl.cu_q).cuda(), wl.seq_lens, wl.cu_q, qv.cuda(), o, ws)
    torch.cuda.synchronize()
    assert mcpu.mcpu_check_device_errors(ws) == 0
    seq = np.repeat(np.arange(wl.batch), wl.q_lens)
    pos = np.concatenate([np.arange(l, l + n) for l, n in zip(wl.seq_lens, wl.q_lens)])
    ref = O.attention(s, seq, pos, qv.double().numpy(), wl.k_pool.float().numpy(), wl.v_pool.float().numpy(),
                      wl.page_table, sinks.numpy())
    PT.check("o", o.float().cpu().double().numpy().reshape(ref.shape), ref, "bf16")
