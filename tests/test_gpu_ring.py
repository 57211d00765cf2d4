"""The direct-to-LDS ring GEMM at the edges of its tiles and of its dispatch:
reductions shorter than the ring, half last units, partial n-tiles, rows just
around a tile, empty and hot groups, rejected scales, both head sizes of the
projection. Tolerances are the layer's (bf16 storage between the products)."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2608_22167_amd import mcpu, workload as W
from tests import parity as PT

pytestmark = pytest.mark.gpu


def _shape(hidden, ffn, fmt="mxfp4", experts=8, top_k=2, **kw):
    return replace(W.GPT_OSS_20B, hidden=hidden, ffn_dim=ffn, n_experts=experts, top_k=top_k, expert_fmt=fmt,
                   **{**dict(n_q_heads=8, n_kv_heads=2, head_dim=64), **kw})


def _forced_moe(s, weights, force, seed):
    T = len(force)
    h = W.synth_normal(seed, 5, (T, s.hidden))
    out = torch.empty((T, s.hidden), device="cuda")
    ws = mcpu.workspace(mcpu.moe_forward_workspace_size(s, T))
    dw = mcpu.DeviceWeights(s, weights)
    mcpu.moe_forward(s, dw, h.cuda(), out, None, None, torch.from_numpy(force).cuda(), ws)
    torch.cuda.synchronize()
    return h, out.cpu().double().numpy(), mcpu.mcpu_check_device_errors(ws)


def _shifted(t, n=4):
    """A copy on the GPU that starts n elements past a 16-byte boundary."""
    buf = torch.empty(t.numel() + n, dtype=t.dtype, device="cuda")
    out = buf[n:].view(t.shape)
    out.copy_(t)
    assert out.data_ptr() % 16 and out.is_contiguous()
    return out


# rows of every eight experts: around 32-row fragments, 64- and 128-row tiles, none, and
# experts holding nearly all (the 12-, 40- and 512-row averages of the dispatch)
ROWS = {"few": [1, 2, 0, 3, 1, 0, 2, 1], "tile64": [31, 32, 33, 63, 64, 0, 65, 24],
        "tile128": [127, 128, 129, 96, 97, 0, 1, 255], "hot": [900, 0, 1, 0, 0, 5, 0, 0], "many": [700, 513, 512, 640, 515, 600, 530, 777]}


@pytest.mark.parametrize("rows", list(ROWS))
# gate/up reductions of 1, 3, 9 and 17 slices and down ones of 5 to 40 (half last units, the
# ring padded and full), 64 .. 5120 columns past whole tiles; 64 experts, so that the work
# is worth the ring
@pytest.mark.parametrize("hidden,ffn", [(64, 2560), (192, 1088), (576, 448), (1088, 320)])
def test_mxfp4_rows_and_reductions(hidden, ffn, rows):
    s = _shape(hidden, ffn, experts=64, top_k=1)
    wl = W.custom(s, [4], [1], 2101 + hidden)
    force = np.random.default_rng(3).permutation(np.repeat(np.arange(64), ROWS[rows] * 8)).astype(np.int32)[:, None]
    h, out, err = _forced_moe(s, wl.weights, force, 11)
    assert err == 0
    T = len(force)
    pick = np.arange(T)
    if T > 400:  # all rows of a few experts, and some of the others
        pick = np.flatnonzero(np.isin(force[:, 0], [6, 34, 63]))
        pick = np.unique(np.concatenate([pick, np.random.default_rng(4).choice(T, 200, replace=False)]))
    ref = O.moe(s, O.Weights(s, wl.weights), h[torch.from_numpy(pick)], force_idx=force[pick])["out"]
    PT.check("moe out", out[pick], ref, "bf16")


# outside the ring: 98 scale blocks per weight row, more than its plan of LDS holds, or scales
# that do not start on 16 bytes; rows per expert of weight slabs (one 64-row item, one and two
# half ones of 128), of 64 x 128, 128 x 128 and 256 x 256 tiles (gate/up; down stays one smaller)
@pytest.mark.parametrize("hidden,rows,shift", [(3136, 12, 0), (3136, 60, 0), (3136, 90, 0), (3136, 120, 0), (3136, 300, 0),
                                               (3136, 700, 0), (1088, 20, 4), (1088, 110, 4)])
def test_mxfp4_beyond_the_ring(hidden, rows, shift):
    s = _shape(hidden, hidden, top_k=1)
    wl = W.custom(s, [4], [1], 2113)
    w = dict(wl.weights)
    if shift:
        for key in ("w_gu_scales", "w_d_scales"):
            w[key] = _shifted(w[key], shift)
    rng = np.random.default_rng(7)
    force = rng.permutation(np.repeat(np.arange(8), rows)).astype(np.int32)[:, None]
    h, out, err = _forced_moe(s, w, force, 16)
    assert err == 0
    pick = np.unique(np.concatenate([[0, len(force) - 1], rng.choice(len(force), 60, replace=False)]))
    ref = O.moe(s, O.Weights(s, wl.weights), h[torch.from_numpy(pick)], force_idx=force[pick])["out"]
    PT.check("moe out", out[pick], ref, "bf16")


@pytest.mark.parametrize("T", [320, 3200])
def test_mxfp4_rejected_scales_contribute_nothing(T):
    """Scales outside [2, 252], anywhere in a tile, raise the error bit, and the
    result is that of the same weights with those blocks' codes zero."""
    s = _shape(576, 576, experts=64)
    wl = W.custom(s, [4], [1], 2111)
    rng = np.random.default_rng(5)
    bad, zero = dict(wl.weights), dict(wl.weights)
    for key in ("w_gu", "w_d"):
        sc, codes = wl.weights[key + "_scales"].clone(), wl.weights[key + "_codes"].clone()
        E, R, B = sc.shape
        for v in (0, 1, 253, 254, 255):
            for _ in range(48):
                e, r, b = int(rng.integers(E)), int(rng.integers(R)), int(rng.integers(B))
                sc[e, r, b] = v
                codes[e, r, 16 * b:16 * b + 16] = 0
        sc[0, 0, 0], sc[-1, -1, -1] = 255, 0
        codes[0, 0, :16], codes[-1, -1, -16:] = 0, 0
        bad[key + "_scales"], zero[key + "_codes"] = sc, codes
    force = rng.integers(0, 64, size=(T, 2)).astype(np.int32)
    _, want, err0 = _forced_moe(s, zero, force, 12)
    _, got, err = _forced_moe(s, bad, force, 12)
    assert err0 == 0 and err & mcpu.DEVERR_MXFP4
    np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("T", [320, 3200, 19200])  # 10, 100 and 600 rows per expert
@pytest.mark.parametrize("key", ["w_gu", "w_d"])
def test_mxfp4_rejected_blocks_are_exactly_zero(key, T):
    """One matrix holds codes 6 in blocks of rejected scales and zeros elsewhere,
    so the experts add exactly nothing. Gate/up: a remainder of 2^-125 would
    come back through down weights of 6 x 2^125. Down: the rows are zero and the
    activations 56 (gate and up biases of 7), so a remainder is the output."""
    s = _shape(576, 576, experts=64)
    wl = W.custom(s, [4], [1], 2112)
    rng = np.random.default_rng(6)
    w = {k: v.clone() for k, v in wl.weights.items()}
    for b in ("b_gu", "b_d"):
        w[b].zero_()
    w["w_d_codes"].fill_(0x77)
    w["w_d_scales"].fill_(252)
    sc, codes = w[key + "_scales"], w[key + "_codes"]
    sc.fill_(120)
    codes.zero_()
    bad = rng.random(tuple(sc.shape)) < 0.05
    bad[:, 0, 0] = bad[:, -1, -1] = True
    sc[torch.from_numpy(bad)] = torch.from_numpy(rng.choice([0, 1, 253, 254, 255], bad.sum()).astype(np.uint8))
    codes[torch.from_numpy(np.repeat(bad, 16, axis=2))] = 0x77
    h = W.synth_normal(14, 5, (T, s.hidden))
    if key == "w_d":
        w["b_gu"].fill_(7.0)
        h.zero_()
    out = torch.full((T, s.hidden), 7.0, device="cuda")
    ws = mcpu.workspace(mcpu.moe_forward_workspace_size(s, T))
    mcpu.moe_forward(s, mcpu.DeviceWeights(s, w), h.cuda(), out, None, None,
                     torch.from_numpy(rng.integers(0, 64, size=(T, 2)).astype(np.int32)).cuda(), ws)
    torch.cuda.synchronize()
    assert mcpu.mcpu_check_device_errors(ws) & mcpu.DEVERR_MXFP4
    assert torch.equal(out.cpu(), h)


@pytest.mark.parametrize("pack", [False, True])
@pytest.mark.parametrize("ffn", [576, 192])
def test_bf16_experts(pack, ffn):
    """64 bf16 groups of 92 rows on average, row-major and streaming-order
    weights: reductions of 17 slices (gate/up), 9 and 3 (down)."""
    s = _shape(1088, ffn, fmt="dense", experts=64, top_k=1)
    wl = W.custom(s, [4], [1], 2121)
    rows = [127, 128, 129, 0, 1, 33, 255, 64] * 8
    force = np.random.default_rng(3).permutation(np.repeat(np.arange(64), rows)).astype(np.int32)[:, None]
    T = len(force)
    h = W.synth_normal(13, 5, (T, s.hidden))
    out = torch.empty((T, s.hidden), device="cuda")
    ws = mcpu.workspace(mcpu.moe_forward_workspace_size(s, T))
    mcpu.moe_forward(s, mcpu.DeviceWeights(s, wl.weights, pack=pack), h.cuda(), out, None, None,
                     torch.from_numpy(force).cuda(), ws)
    torch.cuda.synchronize()
    assert mcpu.mcpu_check_device_errors(ws) == 0
    pick = np.unique(np.concatenate([np.flatnonzero(np.isin(force[:, 0], [0, 2, 4, 63])),
                                     np.random.default_rng(4).choice(T, 300, replace=False)]))
    ref = O.moe(s, O.Weights(s, wl.weights), h[torch.from_numpy(pick)], force_idx=force[pick])["out"]
    PT.check("moe out", out.cpu().double().numpy()[pick], ref, "bf16")


@pytest.mark.parametrize("T", [700, 16384])  # about 88 and 2048 rows per expert: ring and 256 x 256 tiles if aligned
def test_bf16_experts_off_16_byte_boundaries(T):
    """Matrices that direct loads to LDS are not used on."""
    s = _shape(1088, 1088, fmt="dense", top_k=1)
    wl = W.custom(s, [4], [1], 2122)
    w = {k: _shifted(v) if k in ("w_gu", "w_d") else v for k, v in wl.weights.items()}
    dw = mcpu.DeviceWeights(s, w, pack=False)
    assert dw.struct.w_gu % 16 == 8 and dw.struct.w_d % 16 == 8
    force = (np.random.default_rng(4).permutation(T) % 8).astype(np.int32)[:, None]
    h = W.synth_normal(15, 5, (T, s.hidden))
    out = torch.empty((T, s.hidden), device="cuda")
    ws = mcpu.workspace(mcpu.moe_forward_workspace_size(s, T))
    mcpu.moe_forward(s, dw, h.cuda(), out, None, None, torch.from_numpy(force).cuda(), ws)
    torch.cuda.synchronize()
    assert mcpu.mcpu_check_device_errors(ws) == 0
    rows = np.unique(np.concatenate([[0, T - 1], np.random.default_rng(5).choice(T, 90, replace=False)]))
    ref = O.moe(s, O.Weights(s, wl.weights), h[torch.from_numpy(rows)], force_idx=force[rows])["out"]
    PT.check("moe out", out.cpu().double().numpy()[rows], ref, "bf16")


# 128 x 128 tiles above the dispatch's bound for both projections: 64-wide heads
# with a ragged last m-tile, and 32-wide ones (two heads a piece, a partial last n-tile)
@pytest.mark.parametrize("pack", [False, True])
@pytest.mark.parametrize("kw,T", [(dict(hidden=2112, n_q_heads=64, n_kv_heads=8, head_dim=64), 2300),
                                  (dict(hidden=2112, n_q_heads=60, n_kv_heads=6, head_dim=32), 2700)])
def test_projections(kw, T, pack):
    s = _shape(ffn=64, **kw)
    rng = np.random.default_rng(2131)
    wl = W.custom(s, rng.integers(1, 60, size=T), np.ones(T), 2131)
    step = mcpu.DeviceStep(wl)
    step.weights = mcpu.DeviceWeights(s, wl.weights, pack=pack)
    q = torch.empty((T, s.n_q_heads, s.head_dim), dtype=torch.bfloat16, device="cuda")
    o = torch.empty((T, s.attn_dim), dtype=torch.bfloat16, device="cuda")
    h1 = torch.empty((T, s.hidden), device="cuda")
    step.run(mcpu.Taps(q=q.data_ptr(), o=o.data_ptr(), h1=h1.data_ptr()))
    torch.cuda.synchronize()
    assert step.device_errors() == 0
    seqs = sorted({0, 127, 128, T - 1, T - 2} | {int(b) for b in rng.choice(T, 6, replace=False)})
    sub, rows = W.restrict(wl, seqs)
    ref = O.decode_layer(sub)
    for name, got in (("q", q), ("o", o), ("h1", h1)):
        PT.check(name, got[torch.from_numpy(rows).cuda()].float().cpu().double().numpy().reshape(ref[name].shape), ref[name], "bf16")
