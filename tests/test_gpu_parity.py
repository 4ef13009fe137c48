"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the
same seeded inputs.

Tolerances: O max-abs <= 2e-2 (bf16 output); log-sum-exp and importance
<= 1e-3 relative (|a-b| <= 1e-3*max(|b|,1e-6)); index sets exact except at
ties (see check_selection)."""
import os

import numpy as np
import pytest
import torch

import oracle
import workloads as W
import paper_2508_09035_amd as pdd
from gpu_harness import DeviceWorkload, check_selection

pytestmark = pytest.mark.gpu

O_ATOL = 2e-2
REL = 1e-3


def rel_close(got, want, what):
    err = np.abs(got - want)
    tol = REL * np.maximum(np.abs(want), 1e-6)
    bad = err > tol
    assert not bad.any(), (f"{what}: {bad.sum()} of {bad.size} beyond 1e-3 relative; "
                           f"worst ratio {np.max(err / tol):.3g}")


def compare_all(wl, dev, rows=None, label=""):
    O, lse, imp, idx, mask = dev.results()
    window = -1 if wl.chunked else wl.window
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale,
                              rows=rows)
    if rows is not None:
        O, lse = O[rows], lse[:, rows]
    assert np.isfinite(O).all() and np.isfinite(lse).all(), f"{label}: unwritten / non-finite output"
    o_err = np.abs(O - oO).max() if O.size else 0.0
    assert o_err <= O_ATOL, f"{label}: O max-abs error {o_err}"
    rel_close(lse, oL, f"{label} lse")
    if window != 0:
        oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, window)
        assert np.isfinite(imp).all()
        rel_close(imp, oI, f"{label} importance")
        # gate B: GPU scores -> GPU selection vs oracle selection, ties within the score tolerance
        swapped = check_selection(oI, idx, mask, wl, REL, label + " end-to-end select")
        return o_err, swapped
    return o_err, 0


def run_and_compare(wl, rows=None, waves=0, label=""):
    dev = DeviceWorkload(wl)
    dev.poison()
    pdd.set_option(pdd.OPT_ATTN_WAVES, waves)
    try:
        dev.step()
        return compare_all(wl, dev, rows, label or wl.name)
    finally:
        pdd.set_option(pdd.OPT_ATTN_WAVES, 0)


# ----------------------------------------------------------------- small cases
def test_c1_tiny_full():
    wl = W.make_workload("c1")
    _, swapped = run_and_compare(wl)
    assert swapped == 0


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("d", [64, 128])
def test_multi_tile_ragged_gqa(d, waves):
    # several q tiles and key tiles, ragged tails, a 1-token prompt, window > a prompt
    wl = W.make_custom("t", [300, 77, 1, 513, 64, 31], None, 4, 2, d, 40, "3/10", seed=100 + d)
    run_and_compare(wl, waves=waves, label=f"ragged d={d} w={waves}")


@pytest.mark.parametrize("waves", [4, 8])
def test_chunked_small(waves):
    wl = W.make_custom("t", [70, 33, 256], [70 + 130, 33, 256 + 700], 8, 2, 128, 0, "1/4",
                       seed=7, chunked=True)
    wl.cand_end[1] = 0  # a chunk with no prefix: nothing to select
    wl.k_keep[1] = 0
    run_and_compare(wl, waves=waves, label=f"chunked w={waves}")


@pytest.mark.parametrize("seed", range(12))
def test_random_shapes(seed):
    """Seeded random small problems: batch, lengths around the 64-key tile and 256-row
    workgroup boundaries, head grouping, head_dim, window, plain or chunked."""
    rng = np.random.default_rng(1000 + seed)
    B = int(rng.integers(1, 5))
    edges = np.array([1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 255, 256, 257, 320, 511, 512, 513, 700])
    lens_q = [int(rng.choice(edges)) if rng.random() < 0.6 else int(rng.integers(1, 700)) for _ in range(B)]
    hq, hkv = [(1, 1), (4, 1), (4, 2), (8, 8), (6, 2), (8, 2)][int(rng.integers(0, 6))]
    d = int(rng.choice([64, 128]))
    chunked = bool(rng.random() < 0.4)
    if chunked:
        lens_k = [q + (int(rng.choice(edges)) if rng.random() < 0.7 else 0) for q in lens_q]
        wl = W.make_custom("t", lens_q, lens_k, hq, hkv, d, 0, "1/3", seed=seed, chunked=True)
        for b in range(B):                              # a chunk without a prefix has no candidates
            if lens_k[b] == lens_q[b]:
                wl.cand_end[b] = 0
                wl.k_keep[b] = 0
    else:
        wl = W.make_custom("t", lens_q, None, hq, hkv, d, int(rng.integers(1, 100)), "1/3", seed=seed)
    run_and_compare(wl, waves=int(rng.choice([0, 4, 8])),
                    label=f"random {seed}: q={lens_q} chunked={chunked} heads={hq}/{hkv} d={d}")


@pytest.mark.parametrize("d", [64, 128])
def test_short_chunks_behind_a_long_prefix(d):
    """Chunks much shorter than a workgroup (1 to 224 new tokens behind about 5000 keys): most
    waves of a workgroup have no rows and only take part in the K/V requests and the barriers of
    the pipelined and the masked loop; with the library's scratch the importance sweep keeps them
    on the common path.  128 and 256 query rows per workgroup, everything against the oracle."""
    lens_q = [1, 40, 100, 224, 33]
    lens_k = [q + 5000 + 37 * i for i, q in enumerate(lens_q)]
    wl = W.make_custom("t", lens_q, lens_k, 8, 2, d, 0, "1/4", seed=90 + d, chunked=True)
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale)
    oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, -1)
    try:
        for waves in (4, 8):
            pdd.set_option(pdd.OPT_ATTN_WAVES, waves)
            dev = DeviceWorkload(wl)
            for use_ws in (False, True):
                what = f"d={d} waves={waves} scratch={use_ws}"
                dev.poison()
                dev.attn(True, use_workspace=use_ws)
                O, lse, imp = dev.results()[:3]
                assert np.abs(O - oO).max() <= O_ATOL, what + " O"
                rel_close(lse, oL, what + " lse")
                rel_close(imp, oI, what + " importance")
    finally:
        pdd.set_option(pdd.OPT_ATTN_WAVES, 0)


@pytest.mark.parametrize("seed", range(4))
def test_random_chunks_with_long_prefix(seed):
    """Seeded random chunked problems with several query tiles and prefixes of up to 3000 keys, so
    that the importance sweep inside the attention kernel runs its pipelined loop, its masked loop
    and the handover between them; head_dim 64 and 128, 128 and 256 queries per workgroup."""
    rng = np.random.default_rng(7000 + seed)
    B = int(rng.integers(1, 4))
    lens_q = [int(rng.integers(1, 900)) for _ in range(B)]
    lens_k = [q + int(rng.integers(0, 3000)) for q in lens_q]
    hq, hkv = [(4, 1), (8, 2), (16, 2), (8, 8)][int(rng.integers(0, 4))]
    d = int(rng.choice([64, 128]))
    wl = W.make_custom("t", lens_q, lens_k, hq, hkv, d, 0, "1/3", seed=500 + seed, chunked=True)
    for b in range(B):
        if lens_k[b] == lens_q[b]:
            wl.cand_end[b] = 0
            wl.k_keep[b] = 0
    run_and_compare(wl, waves=int(rng.choice([0, 4, 8])),
                    label=f"chunk {seed}: q={lens_q} k={lens_k} heads={hq}/{hkv} d={d}")


_SPLIT_SHAPES = {       # (new tokens, keys or None for prefill, query heads, KV heads, window)
    # groups of 3 heads (rows divide by a number that is no power of two); no queries at all; a key count that
    # is a whole number of tiles; a chunk without prefix
    "group-3": ([1, 0, 33, 127, 3], [5001, 300, 4096, 127, 4], 6, 2, 0),
    "group-16": ([5, 9], [9005, 1033], 16, 1, 0),               # all heads of a token in half a wave
    "mha": ([129, 128, 1], [2629, 6128, 65], 8, 8, 0),         # one row past a row tile and exactly one
    "one-head": ([300], [2500], 1, 1, 0),                       # (at 1500 keys and head_dim 64 the plain form is chosen)
    "prefill": ([3000, 1, 700], None, 2, 1, 40),                # splits that end at the diagonal
}


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("name", list(_SPLIT_SHAPES))
def test_keys_split_over_workgroups(name, d):
    """The attention form that cuts the keys into pieces and packs the heads of a group into its
    tiles, against the oracle on every row; its scratch is filled with NaN patterns before."""
    lens_q, lens_k, hq, hkv, window = _SPLIT_SHAPES[name]
    wl = W.make_custom("t", lens_q, lens_k, hq, hkv, d, window, "1/4", seed=700 + d, chunked=lens_k is not None)
    dev = DeviceWorkload(wl)
    assert dev.workspace_bytes >= 2 * wl.total_q * hq * (d + 1) * 4, "this shape is one that splits its keys"
    dev.poison()
    dev.workspace.fill_(0xFF)
    dev.attn(True)
    torch.cuda.synchronize()
    O, lse, imp = dev.results()[:3]
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale)
    oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, window or -1)
    assert np.abs(O - oO).max() <= O_ATOL
    rel_close(lse, oL, "lse")
    rel_close(imp, oI, "importance")
    assert (dev.workspace.view(torch.int32) != -1).any(), "the scratch was not used"
    bits = [x.clone() for x in (dev.o, dev.lse, dev.imp)]
    dev.poison()
    dev.attn(True)                                              # the same bits again
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(bits, (dev.o, dev.lse, dev.imp)))


@pytest.mark.parametrize("lens,d", [([4000, 130], 128), ([16000, 100], 64)])
def test_prompts_with_their_keys_split(lens, d):
    """Prompts of the key-split form, whose pieces end at the diagonal: rows at the ends of tiles against the oracle."""
    wl = W.make_custom("t", lens, None, 1, 1, d, 0, "1/4", seed=705 + d)
    dev = DeviceWorkload(wl)
    assert dev.attn_form(False) == pdd.ATTN_SPLIT
    dev.poison()
    dev.workspace.fill_(0xFF)
    dev.attn(False)
    O, lse = dev.results()[:2]
    assert np.isfinite(O).all() and np.isfinite(lse).all()
    rows = _wide_rows(wl)
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, rows=rows)
    assert np.abs(O[rows] - oO).max() <= O_ATOL
    rel_close(lse[:, rows], oL, "lse")


@pytest.mark.parametrize("d", [64, 128])
def test_keys_split_over_workgroups_with_a_nan_key(d):
    """A key of NaN, which no caller should pass, spoils the same rows in the same way whichever form runs: every
    row that sees it has NaN outputs and a log-sum-exp of -infinity, and no other row changes."""
    wl = W.make_custom("t", [40, 3], [6000, 2503], 8, 2, d, 0, "1/4", seed=71, chunked=True)
    dev = DeviceWorkload(wl)
    assert dev.workspace_bytes >= 2 * wl.total_q * 8 * (d + 1) * 4, "this shape is one that splits its keys"
    dev.attn(False)
    torch.cuda.synchronize()
    clean = (dev.o.clone(), dev.lse.clone())
    got = []
    for at in (700, 5970):                                      # an early piece, every row; the last one, rows from 10 on
        keep = dev.k[at].clone()
        dev.k[at] = float("nan")
        for scratch in (True, False):
            dev.poison()
            dev.attn(False, use_workspace=scratch)
            torch.cuda.synchronize()
            got.append((dev.o.clone(), dev.lse.clone()))
        dev.k[at] = keep
        (so, sl), (po, pl) = got[-2:]
        first = max(0, at - 5960)
        assert torch.equal(so[:first], clean[0][:first]) and torch.equal(so[40:], clean[0][40:])
        assert torch.isnan(so[first:40]).all() and torch.isnan(po[first:40]).all()
        assert (sl[:, first:40] == -float("inf")).all() and (pl[:, first:40] == -float("inf")).all()
        assert torch.equal(sl[:, :first], clean[1][:, :first]) and torch.equal(sl[:, 40:], clean[1][:, 40:])


_WIDE_SHAPES = {        # (new tokens, keys or None for prefill, query heads, KV heads, head_dim)
    # first tiles of 1, 100 and 255 rows, one row past a tile, whole tiles, an empty sequence, last key tiles of 1 and 64 keys
    "uneven": ([2305, 100, 2561, 1, 255, 0, 257, 2304], None, 16, 4, 128),
    "one prompt": ([2497], None, 32, 8, 128),
    "chunks": ([300, 33, 256, 1, 65], [4300, 4129, 4352, 4031, 65], 64, 8, 128),    # (every row group of a tile 0 missing or there)
    "uneven, 64": ([1100, 1023, 999, 900, 1, 257, 640, 31], None, 64, 8, 64),
    "many, 64": ([600] * 8, None, 32, 8, 64),
}


@pytest.mark.parametrize("lens_q,lens_k", [
    ([2000, 1], None),
    ([1900, 0, 1, 127, 128, 129, 255, 256, 257, 900, 3, 64, 65, 511, 513, 1200], None),     # 16 sequences, as many as are listed
    ([1500, 40, 30], [1500, 9000, 2500]),                               # chunks: keys and queries in other orders; 71 steps of 128
    ([1000, 90, 80, 3], [1000, 8127, 8128, 8131]),                      # the last step of the first 64 and the first of the next
])
def test_tiles_listed_longest_first(lens_q, lens_k):
    """Uneven batches whose workgroups find their tiles among those that exist: every row is written, with the bits of the
    form whose grid holds the longest sequence's tiles for each."""
    wl = W.make_custom("t", lens_q, lens_k, 4, 2, 128, 0, "1/4", seed=880, chunked=lens_k is not None)
    dev = DeviceWorkload(wl)
    got = []
    try:
        for waves, form in ((4, pdd.ATTN_4_WAVES_LISTED), (8, pdd.ATTN_8_WAVES)):
            pdd.set_option(pdd.OPT_ATTN_WAVES, waves)
            assert dev.attn_form(False, use_workspace=False) == form
            dev.poison()
            dev.attn(False, use_workspace=False)
            torch.cuda.synchronize()
            got.append((dev.o.clone(), dev.lse.clone()))
    finally:
        pdd.set_option(pdd.OPT_ATTN_WAVES, 0)
    assert torch.isfinite(got[0][0].float()).all() and torch.isfinite(got[0][1]).all()
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("lens,hq,hkv", [([4000, 900], 16, 8), ([3308, 4000, 5809, 1320, 269], 4, 2)])
def test_tiles_listed_where_the_rule_says_so(lens, hq, hkv):
    """Uneven prompts that the library itself lists the tiles of: rows at the ends of tiles against the oracle."""
    wl = W.make_custom("t", lens, None, hq, hkv, 128, 0, "1/4", seed=881)
    dev = DeviceWorkload(wl)
    assert dev.attn_form(False, use_workspace=False) == pdd.ATTN_4_WAVES_LISTED
    dev.poison()
    dev.attn(False, use_workspace=False)
    O, lse = dev.results()[:2]
    assert np.isfinite(O).all() and np.isfinite(lse).all()
    rows = _wide_rows(wl)
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, rows=rows)
    assert np.abs(O[rows] - oO).max() <= O_ATOL
    rel_close(lse[:, rows], oL, "lse")


def _wide_rows(wl):
    """Rows around the ends of 32-row groups and 256-row tiles, which count from a sequence's end."""
    rows = []
    for b, e in zip(wl.cu_seqlens_q[:-1], wl.cu_seqlens_q[1:]):
        at = [0, 1, 31, 32, 33, 63, 64, 100, 127, 128, 129, 223, 224, 255, 256, 257, 511, 512, e - b - 1]
        rows += [r for x in at for r in (b + x, e - 1 - x) if b <= r < e]
    return np.unique(rows)


@pytest.mark.parametrize("name", list(_WIDE_SHAPES))
def test_wide_attention(name):
    """The form with 64 queries to a wave: selected rows against the oracle, and every row against the form with 32, whose
    sums have the same order: as long as no row's scores rise 8 in log2 above its first 32 keys', the same bits."""
    lens_q, lens_k, hq, hkv, d = _WIDE_SHAPES[name]
    wl = W.make_custom("t", lens_q, lens_k, hq, hkv, d, 0, "1/4", seed=810, chunked=lens_k is not None)
    dev = DeviceWorkload(wl)
    got = []
    try:
        for waves, form in ((0, pdd.ATTN_WIDE), (8, pdd.ATTN_8_WAVES)):
            pdd.set_option(pdd.OPT_ATTN_WAVES, waves)
            assert dev.attn_form(False, use_workspace=False) == form
            dev.poison()
            dev.attn(False, use_workspace=False)
            torch.cuda.synchronize()
            got.append((dev.o.float(), dev.lse.clone()))
    finally:
        pdd.set_option(pdd.OPT_ATTN_WAVES, 0)
    (o, lse), (o8, lse8) = got
    assert torch.isfinite(o).all() and torch.isfinite(lse).all()
    assert torch.equal(o, o8) and torch.equal(lse, lse8)
    rows = _wide_rows(wl)
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, rows=rows)
    assert np.abs(o.cpu().numpy()[rows] - oO).max() <= O_ATOL
    rel_close(lse.cpu().numpy()[:, rows].astype(np.float64), oL, "lse")


@pytest.mark.parametrize("lens_q,lens_k,hq", [
    ([256, 256, 256], [4352, 3840, 2560], 64),             # whole tiles; a step more and a step fewer than whole rounds of the K buffers
    ([200, 1, 256, 97], [4700, 3001, 5000, 3233], 64),      # a tile with rows in half of its waves, hardly any
    ([512, 300, 511], [3712, 3900, 3583], 32),  # two tiles, the first of them with empty groups
])
def test_wide_attention_with_the_importance_sweep(lens_q, lens_k, hq):
    """The sweep behind the form with 64 queries to a wave: importance of every key against the oracle; outputs with the
    bits of attention alone; the same bits again."""
    wl = W.make_custom("t", lens_q, lens_k, hq, 8, 128, 0, "1/4", seed=860, chunked=True)
    dev = DeviceWorkload(wl)
    slices = hq // 8 * ((max(lens_q) + 255) // 256)
    assert dev.workspace_bytes == slices * 8 * wl.total_k * 4, "this shape is one that sweeps"
    assert dev.attn_form() == pdd.ATTN_WIDE
    runs = []
    for _ in range(2):
        dev.poison()
        dev.workspace.fill_(0xFF)
        dev.attn(True)
        runs.append(dev.results()[:3])
    assert all(np.array_equal(a, b) for a, b in zip(*runs))
    O, lse, imp = runs[0]
    rel_close(imp, oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, -1), "importance")
    rows = _wide_rows(wl)
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, rows=rows)
    assert np.abs(O[rows] - oO).max() <= O_ATOL
    rel_close(lse[:, rows], oL, "lse")
    assert np.isfinite(O).all() and np.isfinite(lse).all() and np.isfinite(imp).all()


def test_wide_attention_far_from_its_first_reference_with_the_importance_sweep():
    """The second walk, with a reference that follows the maxima, before the sweep; waves and groups without rows among them.
    One sequence of three rises by 150 behind its first 32 keys."""
    wl = W.make_custom("t", [256, 200, 97], [4700, 3001, 5000], 64, 8, 128, 0, "1/4", seed=861, chunked=True)
    c = np.float32(np.sqrt(150.0 / wl.scale / 128))
    at_q, at_k = np.zeros((wl.total_q, 1, 1), np.float32), np.zeros((wl.total_k, 1, 1), np.float32)
    at_q[wl.cu_seqlens_q[1]:wl.cu_seqlens_q[2]] = 1
    at_k[wl.cu_seqlens_k[1] + 32:wl.cu_seqlens_k[2]] = 1
    wl.q = W.f32_to_bf16_bits(W.bf16_bits_to_f32(wl.q) * 0.5 + c * at_q)
    wl.k = W.f32_to_bf16_bits(W.bf16_bits_to_f32(wl.k) * 0.5 + c * at_k)
    dev = DeviceWorkload(wl)
    assert dev.attn_form() == pdd.ATTN_WIDE
    dev.poison()
    dev.workspace.fill_(0xFF)
    dev.attn(True)
    O, lse, imp = dev.results()[:3]
    assert np.isfinite(O).all() and np.isfinite(lse).all() and np.isfinite(imp).all()
    rel_close(imp, oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, -1), "importance")
    rows = _wide_rows(wl)
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, rows=rows)
    assert np.abs(O[rows] - oO).max() <= O_ATOL
    rel_close(lse[:, rows], oL, "lse")


@pytest.mark.parametrize("layout", ["packed", "head-major"])
@pytest.mark.parametrize("d", [64, 128])
def test_wide_attention_in_other_layouts(d, layout):
    """Views of one QKV buffer and head-major tensors give the bits of the contiguous ones (which the oracle has checked);
    what lies beside the outputs stays."""
    hq, hkv = (64, 8) if d == 64 else (32, 8)
    wl = W.make_custom("t", [2497, 300], None, hq, hkv, d, 0, "1/4", seed=76)
    dev = DeviceWorkload(wl)
    assert dev.attn_form(False) == pdd.ATTN_WIDE
    dev.poison()
    dev.attn(False)
    torch.cuda.synchronize()
    want = [x.clone() for x in (dev.o, dev.lse)]
    beside = torch.zeros((wl.total_q, 2 * hq, d), dtype=torch.bfloat16, device="cuda")
    if layout == "packed":
        qkv = torch.cat((dev.q, dev.k, dev.v), 1)
        dev.q, dev.k, dev.v, dev.o = qkv[:, :hq], qkv[:, hq:hq + hkv], qkv[:, hq + hkv:], beside[:, hq:]
    else:
        dev.q, dev.k, dev.v, dev.o = (x.transpose(0, 1).contiguous().transpose(0, 1) for x in (dev.q, dev.k, dev.v, dev.o))
    assert not dev.q.is_contiguous() and not dev.o.is_contiguous() and dev.attn_form(False) == pdd.ATTN_WIDE
    dev.o.fill_(float("nan"))
    dev.lse.fill_(float("nan"))
    dev.attn(False)
    torch.cuda.synchronize()
    assert torch.equal(dev.o, want[0]) and torch.equal(dev.lse, want[1]) and not beside[:, :hq].any()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("logit,v_exponent", [(150.0, 0), (-150.0, 0), (55.0, 0), (55.0, 100)])
def test_wide_attention_far_from_its_first_reference(logit, v_exponent, d):
    """Keys from 32 on stand far above (below) the first block, which sets the reference: sums beyond 2^100, sums in range
    with 2^-216 beside 1, sums in range but outputs beyond fp32 on the way.  One sequence of two, the other ordinary."""
    hq, hkv, lens = (64, 8, [2400, 300]) if d == 64 else (32, 8, [2400, 300])
    wl = W.make_custom("t", lens, None, hq, hkv, d, 0, "1/4", seed=830 + d)
    c = np.sqrt(abs(logit) / wl.scale / d)
    first = np.arange(wl.total_q) < lens[0]
    wl.q = W.f32_to_bf16_bits(W.bf16_bits_to_f32(wl.q) * 0.5 + np.float32(c) * first[:, None, None])
    at = (np.arange(wl.total_k) >= 32) & first
    wl.k = W.f32_to_bf16_bits(W.bf16_bits_to_f32(wl.k) * 0.5 + np.float32(np.sign(logit) * c) * at[:, None, None])
    wl.v = W.f32_to_bf16_bits(W.bf16_bits_to_f32(wl.v) * np.float32(2.0 ** v_exponent))
    dev = DeviceWorkload(wl)
    assert dev.attn_form(False, use_workspace=False) == pdd.ATTN_WIDE
    dev.poison()
    dev.attn(False, use_workspace=False)
    O, lse = dev.results()[:2]
    rows = _wide_rows(wl)
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, rows=rows)
    assert np.isfinite(O).all() and np.isfinite(lse).all()
    assert np.abs(O[rows] - oO).max() <= O_ATOL * 2.0 ** v_exponent
    rel_close(lse[:, rows], oL, "lse")
    if logit == 55.0 and v_exponent == 0:           # a reference that stays behind shows in the last bits
        try:
            pdd.set_option(pdd.OPT_ATTN_WAVES, 8)
            dev.attn(False, use_workspace=False)
        finally:
            pdd.set_option(pdd.OPT_ATTN_WAVES, 0)
        assert not np.array_equal(O, dev.results()[0]), "this shape is one that takes the other form"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rise,late", [(10.9, range(32, 2400)), (16.0, range(40, 41))])
def test_wide_attention_with_values_near_the_largest(rise, late, d):
    """Values of 2^107 (2^113 at one key), and scores that rise by so much (log2) over the first block at many keys or at one:
    such probabilities times such values, not divided by their sum yet, are beyond fp32, though every part of the sum is small."""
    wl = W.make_custom("t", [2400, 300], None, 64, 8, d, 0, "1/4", seed=3)
    c = np.sqrt(rise * np.log(2.0) / wl.scale / d)
    at = np.isin(np.arange(wl.total_k), list(late))
    wl.q = W.f32_to_bf16_bits(np.full(wl.q.shape, c, dtype=np.float32))
    wl.k = W.f32_to_bf16_bits(np.broadcast_to(np.float32(c) * at[:, None, None], wl.k.shape))
    v = np.full(wl.total_k, 2.0 ** 107)
    if len(late) == 1:
        v[late[0]] = 2.0 ** 113
    wl.v = W.f32_to_bf16_bits(np.broadcast_to(v[:, None, None], wl.v.shape))
    dev = DeviceWorkload(wl)
    assert dev.attn_form(False, use_workspace=False) == pdd.ATTN_WIDE
    dev.poison()
    dev.attn(False, use_workspace=False)
    O = dev.results()[0]
    assert np.isfinite(O).all()
    # all rows of a sequence that see the same number of such keys are averages of the same values; bf16 of O, and of q, k and
    # the probabilities in the second case's weights
    score = np.float64(W.bf16_bits_to_f32(W.f32_to_bf16_bits(np.array([c], np.float32)))[0]) ** 2 * d * wl.scale
    w = np.where(at, np.exp(score), 1.0)
    for b, e in ((0, 2400), (2400, 2700)):
        want = np.cumsum(w[b:e] * v[b:e]) / np.cumsum(w[b:e])
        assert np.abs(O[b:e] / want[:, None, None] - 1.0).max() <= 2.0 ** -7


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens_q,lens_k", [([2400, 300], None), ([300, 2048], [4300, 5000])])
def test_wide_attention_without_a_score_in_the_first_block(lens_q, lens_k, d):
    """The first 32 keys' products with every query leave fp32 (scores of -inf); the others lie near -150.  Rows that see one of
    those are as if the first 32 keys did not exist."""
    wl = W.make_custom("t", lens_q, lens_k, 64, 8, d, 0, "1/4", seed=5, chunked=lens_k is not None)
    first = np.zeros(wl.total_k, dtype=bool)
    for b in wl.cu_seqlens_k[:-1]:
        first[b:b + 32] = True
    wl.q = W.f32_to_bf16_bits(np.full(wl.q.shape, 2.0 ** 60, dtype=np.float32))
    k = -2.0 ** -60 * (150.0 / (wl.scale * d) + 0.1 * W.bf16_bits_to_f32(wl.k).astype(np.float64))
    wl.k = W.f32_to_bf16_bits(np.where(first[:, None, None], -2.0 ** 70, k).astype(np.float32))
    dev = DeviceWorkload(wl)
    assert (dev.attn_form(False, use_workspace=False) == pdd.ATTN_WIDE) == (lens_k is None or d == 128)
    dev.poison()
    dev.attn(False, use_workspace=False)
    O, lse = dev.results()[:2]
    rows = _wide_rows(wl)
    at, seq = rows - wl.cu_seqlens_q[np.searchsorted(wl.cu_seqlens_q, rows, "right") - 1], np.searchsorted(wl.cu_seqlens_q, rows, "right") - 1
    rows = rows[at + (wl.seqlens_k - wl.seqlens_q)[seq] >= 32]
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, rows=rows)
    assert np.abs(O[rows] - oO).max() <= O_ATOL
    rel_close(lse[:, rows], oL, "lse")


@pytest.mark.parametrize("lens_q,lens_k,hq,d", [([2400, 300], None, 32, 128), ([2400, 300], None, 64, 64), ([300, 256], [4300, 5000], 64, 128)])
@pytest.mark.parametrize("gain,heavy", [(1, 0), (4, 0), (8, 0), (16, 0), (4, 6), (16, 6)])
def test_wide_attention_is_as_exact_as_the_form_with_32_queries(lens_q, lens_k, hq, d, gain, heavy):
    """Sharp scores, whose largest probabilities do not lie close to the first reference's 1: O no further from 64 bits (in
    the 2-norm over every 16th row, 8e5 values and more, whose errors differ between the forms by 1e-3 of it; a sum that
    leaves out what the probabilities lose to bf16 shows as 0.08 and more at gain 4)."""
    wl = W.make_custom("t", lens_q, lens_k, hq, 8, d, 0, "1/4", seed=890 + d, chunked=lens_k is not None)
    rng = np.random.default_rng(5)
    wl.q = W.f32_to_bf16_bits(W.bf16_bits_to_f32(wl.q) * np.float32(gain))
    k = W.bf16_bits_to_f32(wl.k).copy()
    u = rng.standard_normal((8, d)).astype(np.float32)
    at = rng.permutation(wl.total_k)[:wl.total_k // 100]
    k[at] += heavy * u / np.linalg.norm(u, axis=1, keepdims=True)
    wl.k = W.f32_to_bf16_bits(k)
    rows = np.arange(0, wl.total_q, 16)
    oO = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, rows=rows)[0]
    dev = DeviceWorkload(wl)
    err = []
    try:
        for waves, form in ((0, pdd.ATTN_WIDE), (8, pdd.ATTN_8_WAVES)):
            pdd.set_option(pdd.OPT_ATTN_WAVES, waves)
            assert dev.attn_form(False, use_workspace=False) == form
            dev.poison()
            dev.attn(False, use_workspace=False)
            err.append(np.linalg.norm(dev.results()[0][rows] - oO) / np.linalg.norm(oO))
    finally:
        pdd.set_option(pdd.OPT_ATTN_WAVES, 0)
    print(f"O against 64 bits, gain {gain} heavy {heavy} d {d}: 64 queries {err[0]:.3e}, 32 queries {err[1]:.3e}")
    assert err[0] <= 1.01 * err[1]


@pytest.mark.parametrize("d", [64, 128])
def test_wide_attention_with_a_nan_key(d):
    """A key of NaN spoils the rows that see it (NaN outputs, log-sum-exp -infinity) and no others."""
    wl = W.make_custom("t", [2400, 300], None, 64, 8, d, 0, "1/4", seed=77)
    dev = DeviceWorkload(wl)
    assert dev.attn_form(False, use_workspace=False) == pdd.ATTN_WIDE
    dev.attn(False, use_workspace=False)
    torch.cuda.synchronize()
    clean = (dev.o.float(), dev.lse.clone())
    for at in (5, 1300, 2399):
        keep = dev.k[at].clone()
        dev.k[at] = float("nan")
        dev.poison()
        dev.attn(False, use_workspace=False)
        torch.cuda.synchronize()
        dev.k[at] = keep
        o, lse = dev.o.float(), dev.lse
        assert torch.isnan(o[at:2400]).all() and (lse[:, at:2400] == -float("inf")).all()
        for part in (slice(0, at), slice(2400, None)):
            assert (o[part] - clean[0][part]).abs().max().item() <= O_ATOL
            assert (lse[:, part] - clean[1][:, part]).abs().max().item() <= 1e-5


def test_empty_sequence_in_batch_and_no_host_copies():
    wl = W.make_custom("t", [40, 0, 129], None, 2, 1, 64, 16, "1/2", seed=9)
    dev = DeviceWorkload(wl)
    dev.poison()
    dev.attn(True, host_cu=False)
    dev.select()
    compare_all(wl, dev, label="empty-seq")


def test_mha_and_large_group():
    run_and_compare(W.make_custom("t", [200], None, 3, 3, 128, 200, "1/2", seed=12), label="mha")
    run_and_compare(W.make_custom("t", [150], None, 16, 1, 64, 8, "1/10", seed=13), label="g16")


def test_strided_views_of_a_packed_qkv_buffer():
    wl = W.make_custom("t", [333], None, 4, 2, 128, 32, "1/2", seed=21)
    dev = DeviceWorkload(wl)
    n, hq, hkv, d = 333, 4, 2, 128
    packed = torch.zeros((n, hq + 2 * hkv, d), dtype=torch.bfloat16, device="cuda")
    packed[:, :hq] = dev.q
    packed[:, hq:hq + hkv] = dev.k
    packed[:, hq + hkv:] = dev.v
    dev.q, dev.k, dev.v = packed[:, :hq], packed[:, hq:hq + hkv], packed[:, hq + hkv:]
    dev.poison()
    dev.step()
    compare_all(wl, dev, label="strided")


@pytest.mark.parametrize("layout", ["packed", "head-major"])
@pytest.mark.parametrize("d", [64, 128])
def test_keys_split_over_workgroups_in_other_layouts(d, layout):
    """The key-split form packs the heads of a group into its tiles with the head strides of Q and O: views of one
    QKV buffer, and head-major tensors, give the bits of the contiguous ones (which the oracle has checked)."""
    wl = W.make_custom("t", [40, 0, 3], [6000, 70, 2503], 6, 2, d, 0, "1/4", seed=75, chunked=True)
    dev = DeviceWorkload(wl)
    assert dev.workspace_bytes >= 2 * wl.total_q * 6 * (d + 1) * 4, "this shape is one that splits its keys"
    dev.poison()
    dev.attn(True)
    torch.cuda.synchronize()
    want = [x.clone() for x in (dev.o, dev.lse, dev.imp)]
    if layout == "packed":              # queries and outputs side by side per token, keys and values likewise
        qo = torch.zeros((wl.total_q, 12, d), dtype=torch.bfloat16, device="cuda")
        kv = torch.zeros((wl.total_k, 4, d), dtype=torch.bfloat16, device="cuda")
        qo[:, :6], kv[:, :2], kv[:, 2:] = dev.q, dev.k, dev.v
        dev.q, dev.o, dev.k, dev.v = qo[:, :6], qo[:, 6:], kv[:, :2], kv[:, 2:]
    else:
        dev.q, dev.k, dev.v, dev.o = (x.transpose(0, 1).contiguous().transpose(0, 1) for x in (dev.q, dev.k, dev.v, dev.o))
    assert not dev.q.is_contiguous() and not dev.o.is_contiguous()
    dev.o.fill_(float("nan"))
    dev.lse.fill_(float("nan"))
    dev.imp.fill_(float("nan"))
    dev.workspace.fill_(0xFF)
    dev.attn(True)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(want, (dev.o, dev.lse, dev.imp)))


_ROWS_SHAPES = {        # (new tokens, keys or None for prefill, query heads, KV heads, partial rows in scratch)
    # a workgroup to a tile of 32 rows: around a row tile, a block and a key tile; no keys shared by two heads
    "whole prompts": ([1, 31, 32, 33, 64, 65, 500], None, 1, 1, False),
    "whole, group 3": ([1, 33, 40, 0, 11], [200, 33, 300, 7, 65], 6, 2, False),
    # keys divided, 32 rows: more sequences than lanes, an empty one; more heads in a group than rows in a tile
    "many short": ([1] * 69 + [0, 1], [400 + 37 * i for i in range(69)] + [90, 6000], 6, 2, True),
    "group 48": ([3, 1], [4003, 2500], 48, 1, True),
    # keys divided, 128 rows: around a row tile (at head_dim 64 the second one takes 32 rows); more sequences than lanes
    "chunks": ([43, 0, 1, 85, 300], [3043, 70, 4001, 5085, 3300], 12, 2, True),
    "mha": ([32, 33, 31, 129, 127, 128], [5032, 4033, 6031, 6128, 3000, 6144], 8, 8, True),
    "many chunks": ([6] * 66 + [0, 43], [300 + 30 * i for i in range(66)] + [50, 4000], 36, 1, True),
}


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("name", list(_ROWS_SHAPES))
def test_few_rows_over_many_keys(name, d):
    """The attention forms that share a row tile's keys out over the waves of a workgroup, and over workgroups,
    against the oracle on every row with the scratch full of NaN patterns; then the same bits from views with
    strides, without the host's copy of the lengths."""
    lens_q, lens_k, hq, hkv, divided = _ROWS_SHAPES[name]
    window = 16 if lens_k is None else 0
    wl = W.make_custom("t", lens_q, lens_k, hq, hkv, d, window, "1/4", seed=720 + d, chunked=lens_k is not None)
    dev = DeviceWorkload(wl)
    row_bytes = wl.total_q * hq * (d + 1) * 4
    assert (dev.workspace_bytes >= row_bytes + row_bytes // 4) == divided, "this shape is one that takes the form"
    bits = []
    for views in (False, True):
        if views:
            qo = torch.zeros((wl.total_q, 2 * hq, d), dtype=torch.bfloat16, device="cuda")
            kv = torch.zeros((wl.total_k, 2 * hkv, d), dtype=torch.bfloat16, device="cuda")
            qo[:, :hq], kv[:, :hkv], kv[:, hkv:] = dev.q, dev.k, dev.v
            dev.q, dev.o, dev.k, dev.v = qo[:, :hq], qo[:, hq:], kv[:, :hkv], kv[:, hkv:]
        dev.o.fill_(float("nan"))
        dev.lse.fill_(float("nan"))
        dev.imp.fill_(float("nan"))
        if dev.workspace is not None:
            dev.workspace.fill_(0xFF)
        dev.attn(True, host_cu=not views)
        torch.cuda.synchronize()
        bits.append([x.clone() for x in (dev.o, dev.lse, dev.imp)])
        if not views:
            O, lse, imp = dev.results()[:3]
            assert not divided or (dev.workspace.view(torch.int32) != -1).any(), "the scratch was not used"
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale)
    assert np.abs(O - oO).max() <= O_ATOL
    rel_close(lse, oL, "lse")
    rel_close(imp, oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, window or -1), "importance")
    assert all(torch.equal(a, b) for a, b in zip(*bits))
    if not divided:                     # the form whose waves walk all keys of their own rows rounds elsewhere
        try:
            pdd.set_option(pdd.OPT_ATTN_WAVES, 4)
            dev.attn(True)
            torch.cuda.synchronize()
        finally:
            pdd.set_option(pdd.OPT_ATTN_WAVES, 0)
        assert not torch.equal(dev.o, bits[1][0]), "this shape is one that takes the form"
        assert np.abs(dev.results()[0] - oO).max() <= O_ATOL


@pytest.mark.parametrize("d,name", [(128, "chunks"), (64, "many short"), (64, "mha")])
def test_keys_divided_over_less_scratch(d, name):
    """Scratch smaller than the call asks for: the keys are divided into fewer pieces, down to room for 5/4 partial rows
    for every row beside the table of the rows' pieces; the bytes behind it are left alone."""
    lens_q, lens_k, hq, hkv, _ = _ROWS_SHAPES[name]
    wl = W.make_custom("t", lens_q, lens_k, hq, hkv, d, 0, "1/4", seed=750 + d, chunked=True)
    dev = DeviceWorkload(wl)
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale)
    table, row = wl.total_q * hq * 16, hq * (d + 1) * 4
    least = table + row * (wl.total_q + (wl.total_q + 3) // 4)
    assert least < dev.workspace_bytes // 2
    dev.attn(False, use_workspace=False)
    torch.cuda.synchronize()
    plain = dev.o.clone()
    for size in (dev.workspace_bytes, dev.workspace_bytes - 4, dev.workspace_bytes // 2 // 16 * 16 + 8, least, least - 4):
        dev.poison()
        dev.workspace.fill_(0xFF)
        dev.attn(False, use_workspace=size)
        O, lse = dev.results()[:2]
        assert np.abs(O - oO).max() <= O_ATOL, size
        rel_close(lse, oL, f"lse, {size} bytes")
        assert (dev.workspace[size:] == 0xFF).all()
        if size >= dev.workspace_bytes // 2:
            assert (dev.workspace[:size] != 0xFF).any(), size
        if size < least:
            assert torch.equal(dev.o, plain)


@pytest.mark.parametrize("d,name", [(128, "chunks"), (64, "many short")])
def test_tokens_of_no_sequence_keep_their_outputs(d, name):
    """Lengths on the device that begin behind the first tokens and end before the last ones, on the scratch of a call
    whose lengths covered all: the outputs of tokens outside stay as they are, the others are the earlier call's."""
    lens_q, lens_k, hq, hkv, _ = _ROWS_SHAPES[name]
    wl = W.make_custom("t", lens_q, lens_k, hq, hkv, d, 0, "1/4", seed=740 + d, chunked=True)
    dev = DeviceWorkload(wl)
    dev.attn(False)
    torch.cuda.synchronize()
    want = dev.o.clone(), dev.lse.clone()
    first, end = lens_q[0], wl.total_q - lens_q[-1]
    for cu, lens in ((dev.cu_q, lens_q), (dev.cu_k, lens_k)):
        cu[0] = lens[0]                                           # the first sequence is empty
        cu[-1] -= lens[-1]                                        # and so is the last one
    dev.o.fill_(7.0)
    dev.lse.fill_(7.0)
    dev.attn(False, host_cu=False)
    torch.cuda.synchronize()
    for rest in (slice(0, first), slice(end, None)):
        assert (dev.o[rest] == 7.0).all() and (dev.lse[:, rest] == 7.0).all()
    # (the pieces may be others, whose probabilities round to bf16 at other places)
    assert (dev.o[first:end].float() - want[0][first:end].float()).abs().max() <= O_ATOL
    assert torch.allclose(dev.lse[:, first:end], want[1][:, first:end], rtol=REL)


_LOW_SHAPES = {         # (new tokens, keys or None for prefill, query heads, KV heads, waves, scratch)
    "whole prompt": ([70, 500], None, 1, 1, 0, False),
    "whole chunk": ([1, 40], [200, 300], 4, 2, 0, False),
    "divided, 32 rows": ([1] * 8, [600 + 777 * i for i in range(8)], 32, 8, 0, True),
    "divided, 128 rows": ([43, 85, 300], [3043, 5085, 3300], 12, 2, 0, True),
    "key split": ([6000], None, 2, 1, 0, True),
    "plain, 4 waves": ([70, 500], None, 2, 1, 4, False),
    "plain, 8 waves": ([70, 500], None, 2, 1, 8, False),
    "sweep": ([256, 200], [1256, 900], 4, 2, 8, True),
}


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("name", list(_LOW_SHAPES))
def test_logits_far_below_zero(name, d):
    """Keys that stand against every query: scaled logits near -150, where e^-logit is beyond fp32 before a row has a
    reference.  All keys; keys 32 to 63 alone; all but a sequence's last one.  Every form, against the oracle."""
    lens_q, lens_k, hq, hkv, waves, scratch = _LOW_SHAPES[name]
    window = 32 if lens_k is None else 0
    wl = W.make_custom("t", lens_q, lens_k, hq, hkv, d, window, "1/4", seed=760 + d, chunked=lens_k is not None)
    c = np.sqrt(150.0 / wl.scale / d)                             # of each of the d components
    wl.q = W.f32_to_bf16_bits(W.bf16_bits_to_f32(wl.q) * 0.5 + np.float32(c))
    ordinary = W.bf16_bits_to_f32(wl.k) * 0.5
    local = np.concatenate([np.arange(n) for n in wl.seqlens_k])
    last = np.concatenate([np.arange(n) == n - 1 for n in wl.seqlens_k])
    rows = np.unique(np.concatenate([np.r_[b, min(b + 40, e - 1), max(b, e - 33):e]
                                     for b, e in zip(wl.cu_seqlens_q[:-1], wl.cu_seqlens_q[1:])]))
    try:
        pdd.set_option(pdd.OPT_ATTN_WAVES, waves)
        for which, low in (("all", local >= 0), ("a block", (local >= 32) & (local < 64)), ("all but the last", ~last)):
            wl.k = W.f32_to_bf16_bits(ordinary - np.float32(c) * low[:, None, None])
            dev = DeviceWorkload(wl)
            dev.poison()
            dev.attn(True, use_workspace=scratch)
            O, lse, imp = dev.results()[:3]
            oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, rows=rows)
            oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, window or -1)
            assert np.isfinite(O).all() and np.isfinite(lse).all() and np.isfinite(imp).all(), which
            assert np.abs(O[rows] - oO).max() <= O_ATOL, which
            rel_close(lse[:, rows], oL, which + " lse")
            rel_close(imp, oI, which + " importance")
    finally:
        pdd.set_option(pdd.OPT_ATTN_WAVES, 0)


@pytest.mark.parametrize("lens_q,lens_k,hq,hkv,scratch", [
    ([3000], None, 1, 1, True),                              # key split: 32 rows per wave
    ([40, 200], None, 2, 2, False),                          # whole, 32 rows
    ([40], [4000], 4, 2, True),                              # divided, 32 rows
])
def test_query_rows_sixteen_mebibytes_apart(lens_q, lens_k, hq, hkv, scratch):
    """Q rows 2^23 elements apart are beyond what 128 rows can address with 32 bits, not what 32 rows can: the forms
    that address 32 take them, with the bits of the packed layout and not those of the plain form."""
    wl = W.make_custom("t", lens_q, lens_k, hq, hkv, 64, 0, "1/4", seed=24, chunked=lens_k is not None)
    dev = DeviceWorkload(wl)
    packed, far = dev.q, torch.empty_strided((wl.total_q, hq, 64), (1 << 23, 64, 1), dtype=torch.bfloat16, device="cuda")
    far.copy_(packed)
    got = []
    try:
        for dev.q, waves in ((packed, 4), (packed, 0), (far, 0)):
            pdd.set_option(pdd.OPT_ATTN_WAVES, waves)
            dev.poison()
            dev.attn(False, use_workspace=scratch)
            torch.cuda.synchronize()
            got.append((dev.o.clone(), dev.lse.clone()))
    finally:
        pdd.set_option(pdd.OPT_ATTN_WAVES, 0)
    assert not torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[1][0], got[2][0]) and torch.equal(got[1][1], got[2][1])


def test_rows_a_mebibyte_apart_close_to_the_4_gib_span_limit():
    """Q, K and V rows 1 MiB apart (views into 3.1 GiB buffers): byte offsets inside the sequence's
    span run up to 3.4 * 2^30, close to what 32-bit buffer offsets can address; same bits as
    the packed layout, in the key-split form (with scratch) and in the plain one (without).  With the rows
    1.25 MiB apart the span passes the limit and the call is refused on the host."""
    n, hq, hkv, d = 3000, 4, 2, 128
    wl = W.make_custom("t", [n], None, hq, hkv, d, 64, "1/2", seed=23)
    dev = DeviceWorkload(wl)

    def both_forms():
        got = []
        for scratch in (True, False):
            dev.poison()
            dev.attn(True, use_workspace=scratch)
            dev.select()
            torch.cuda.synchronize()
            got.append([x.clone() for x in (dev.o, dev.lse, dev.imp, dev.idx, dev.mask)])
        return got

    want = both_forms()
    assert not torch.equal(want[0][0], want[1][0]), "with scratch this shape splits its keys"
    row = 1 << 19                                            # elements between rows = 1 MiB
    bufs = []
    for name, heads in (("k", hkv), ("v", hkv), ("q", hq)):       # Q too: the importance kernel addresses it like that
        big = torch.empty((n - 1) * row + heads * d, dtype=torch.bfloat16, device="cuda")
        view = torch.as_strided(big, (n, heads, d), (row, d, 1))
        view.copy_(getattr(dev, name))
        setattr(dev, name, view)
        bufs.append(big)
    for form, a, b in zip(("key split", "plain"), want, both_forms()):
        for what, x, y in zip(("O", "lse", "importance", "indices", "mask"), a, b):
            assert torch.equal(x, y), f"{form}: {what}"
    # (3000 + 512) rows x 1 MiB stays below 4 GiB; with rows 1.25 MiB apart it does not
    wrow = row + (row >> 2)
    del bufs
    wide_buf = torch.empty((n - 1) * wrow + hkv * d, dtype=torch.bfloat16, device="cuda")
    wide = torch.as_strided(wide_buf, (n, hkv, d), (wrow, d, 1))
    with pytest.raises(Exception, match="4 GiB"):
        pdd.prefill_attn(dev.q, wide, dev.v, dev.o, dev.lse, dev.imp, dev.cu_q, dev.cu_k,
                         dev.max_q, dev.max_k, wl.scale, wl.window)
    # a wave addresses its 32 rows of Q the same way: rows 128 MiB apart are refused as well
    del wide, wide_buf
    wl2 = W.make_custom("t", [2], None, hq, hkv, d, 1, "1/2", seed=24)
    dev2 = DeviceWorkload(wl2)
    q_buf = torch.empty((1 << 26) + hq * d, dtype=torch.bfloat16, device="cuda")
    q_wide = torch.as_strided(q_buf, (2, hq, d), (1 << 26, d, 1))
    with pytest.raises(Exception, match="32 rows of Q"):
        pdd.prefill_attn(q_wide, dev2.k, dev2.v, dev2.o, dev2.lse, dev2.imp, dev2.cu_q, dev2.cu_k,
                         dev2.max_q, dev2.max_k, wl2.scale, wl2.window)


def test_two_streams_at_once_with_separate_scratch():
    """The whole path of two different problems enqueued on two streams (default priority) at the
    same time, each with its own outputs and scratch: the bits of the runs one after the other."""
    wls = [W.make_custom("t", [256, 200], [256 + 3000, 200 + 2500], 16, 2, 128, 0, "1/4", seed=61, chunked=True),
           W.make_custom("t", [1500, 700], None, 8, 2, 128, 64, "1/3", seed=62)]
    devs = [DeviceWorkload(wl) for wl in wls]
    want = []
    for dev in devs:
        dev.poison()
        dev.step()
        torch.cuda.synchronize()
        want.append([x.clone() for x in (dev.o, dev.lse, dev.imp, dev.idx, dev.mask)])
        dev.poison()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for _ in range(3):                                      # interleaved enqueues, several rounds
        for dev, st in zip(devs, streams):
            with torch.cuda.stream(st):
                dev.step()
    torch.cuda.synchronize()
    for dev, w in zip(devs, want):
        for what, a, b in zip(("O", "lse", "importance", "indices", "mask"), w,
                              (dev.o, dev.lse, dev.imp, dev.idx, dev.mask)):
            assert torch.equal(a, b), what


@pytest.mark.parametrize("lens,heads,window,streams", [([700, 90], (8, 2), 64, False),
                                                       ([300, 97, 64, 1023], (6, 2), 203, True)])
def test_standalone_importance_equals_fused_and_is_deterministic(lens, heads, window, streams):
    """The standalone call against the one behind the attention, with and without scratch: window rows that fit
    the LDS (which need none), and longer windows in the streaming kernel, whose rows are divided over workgroups
    where there is scratch."""
    wl = W.make_custom("t", lens, None, *heads, 128, window, "1/2", seed=31)
    dev = DeviceWorkload(wl)
    desc, keep = pdd.make_desc(dev.q, dev.k, None, None, dev.cu_q, dev.cu_k, dev.max_q, dev.max_k, wl.scale, wl.window)
    need = pdd.workspace_bytes(desc, pdd.CALL_TOKEN_IMPORTANCE)
    del keep
    assert (need > 0) == streams and dev.workspace_bytes >= need
    dev.poison()
    dev.step()
    O1, l1, i1, x1, m1 = dev.results()
    imp2 = torch.full_like(dev.imp, float("nan"))
    if streams:
        dev.workspace.fill_(0xFF)
    pdd.token_importance(dev.q, dev.k, dev.lse, imp2, dev.cu_q, dev.cu_k, dev.max_q, dev.max_k,
                         wl.scale, wl.window, wl.cu_seqlens_q, wl.cu_seqlens_k, workspace=dev.workspace)
    torch.cuda.synchronize()
    assert np.array_equal(imp2.cpu().numpy(), dev.imp.cpu().numpy())
    assert not streams or (dev.workspace != 0xFF).any(), "the scratch was not used"
    # without scratch the single-pass form runs: same values up to the order of the fp32 additions
    imp3 = torch.full_like(dev.imp, float("nan"))
    pdd.token_importance(dev.q, dev.k, dev.lse, imp3, dev.cu_q, dev.cu_k, dev.max_q, dev.max_k,
                         wl.scale, wl.window, wl.cu_seqlens_q, wl.cu_seqlens_k)
    torch.cuda.synchronize()
    np.testing.assert_allclose(imp3.cpu().numpy(), dev.imp.cpu().numpy(), rtol=1e-5, atol=1e-12)
    oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, wl.window)
    rel_close(imp2.cpu().numpy().astype(np.float64), oI, "importance")
    rel_close(imp3.cpu().numpy().astype(np.float64), oI, "importance without scratch")
    dev.poison()
    dev.step()
    O2, l2, i2, x2, m2 = dev.results()
    assert np.array_equal(O1, O2) and np.array_equal(l1, l2) and np.array_equal(i1, i2)
    assert np.array_equal(x1, x2) and np.array_equal(m1, m2)
    # attention without importance leaves the importance buffer alone
    dev.imp.fill_(-5.0)
    dev.attn(with_importance=False)
    torch.cuda.synchronize()
    assert (dev.imp == -5.0).all()


@pytest.mark.parametrize("name", ["c5", "chunk-ragged", "chunk-tiles", "chunk-d64"])
def test_importance_with_and_without_scratch(name):
    """The three forms of the importance step in chunked mode, each against the oracle: as a
    second sweep inside the attention kernel (all of the scratch the library asks for, both head
    dimensions), as the separate kernel with its window rows divided over several workgroups or in
    a single pass (one byte less than that: whatever still fits), and without any scratch.
    Partial sums live in the caller's scratch and are added in a fixed order."""
    if name == "c5":
        wl = W.make_workload(name)
    elif name == "chunk-ragged":   # ragged chunks with 16 query heads per KV head
        wl = W.make_custom("t", [200, 256, 77, 256], [200 + 9000, 256 + 7000, 77 + 8000, 256 + 8100], 32, 2, 128, 0,
                           "1/4", seed=41, chunked=True)
    elif name == "chunk-tiles":    # chunks of several 256-row query tiles; one without queries (its keys
        # must come out as zeros), one without a prefix, one of a single row
        wl = W.make_custom("t", [700, 0, 513, 256, 1], [700 + 1500, 300, 513, 256 + 64, 1 + 900], 8, 2, 128, 0,
                           "1/4", seed=43, chunked=True)
    else:                          # head_dim 64
        wl = W.make_custom("t", [256, 200, 256, 256], [256 + 8000, 200 + 9000, 256 + 8100, 256 + 7000], 32, 2, 64, 0,
                           "1/4", seed=47, chunked=True)
    oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, -1 if wl.chunked else wl.window)
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale) if name == "chunk-tiles" else (None, None)
    try:
        for waves in ((4, 8) if name == "chunk-tiles" else (0,)):      # 128 and 256 query rows per workgroup
            pdd.set_option(pdd.OPT_ATTN_WAVES, waves)
            dev = DeviceWorkload(wl)                                     # sizes its scratch for this option
            assert dev.workspace_bytes > 0
            for use_ws in (True, dev.workspace_bytes - 1, False):
                what = f"{name} waves={waves} scratch={use_ws}"
                dev.poison()
                dev.workspace.fill_(0xFF)   # NaN patterns: a partial sum that is not overwritten shows
                dev.attn(True, use_workspace=use_ws)
                torch.cuda.synchronize()
                rel_close(dev.imp.cpu().numpy().astype(np.float64), oI, what + " importance")
                if oO is not None:          # the sweep must leave the attention output alone
                    O, lse = dev.results()[:2]
                    assert np.abs(O - oO).max() <= O_ATOL, what + " O"
                    rel_close(lse, oL, what + " lse")
    finally:
        pdd.set_option(pdd.OPT_ATTN_WAVES, 0)


@pytest.mark.parametrize("lens,prefix,hq,hkv,d,window", [
    ([31, 1, 0, 33, 500], None, 4, 4, 64, 1),                     # one row; sequences of a key and of none
    ([513, 700], None, 10, 2, 128, 13),                           # 65 rows of 5 heads
    ([300, 97, 64, 1023], None, 6, 2, 128, 200),                  # windows longer than some of the prompts, 600 rows: 19 blocks
    ([300, 97, 64, 1023], None, 6, 2, 128, 203),                  # 20 blocks: the streaming kernel
    ([1000, 1300], None, 8, 2, 64, 300),                          # 1200 rows of head_dim 64: the streaming kernel
    ([7, 0, 1, 40], [900, 77, 2049, 1500], 6, 2, 128, -1),        # chunks, one without tokens: its keys read zero
    ([9, 30], [6000, 3100], 16, 16, 64, -1),                      # one block of rows: four waves, two key groups each
    ([9, 40], [6000, 3100], 16, 16, 64, -1),                      # two: eight waves, two key groups each
    ([64], [8161], 128, 16, 128, -1),                             # sixteen waves, one key group each, 512 rows
    ([64], [16320], 128, 16, 128, -1),                            # sixteen waves, two key groups each
    # sequences of different lengths, whose workgroups look up their pieces: sixteen waves of two groups; four of one
    ([64, 20, 3], [3, 2500, 9990], 128, 16, 128, -1),
    ([17, 0, 5, 40], [900, 70, 5000, 1500], 32, 8, 64, -1),
    ([1] * 63 + [9, 3], list(range(65)), 32, 8, 64, -1),          # 65 sequences: more than are looked up
    # the streaming kernel over sequences of different lengths: slices looked up, rows divided; 65 sequences: not looked up
    ([3, 200, 0, 31], [4000, 500, 100, 77], 16, 4, 128, -1),
    ([2] * 62 + [170, 0, 9], list(range(65)), 16, 2, 128, -1),
    ([300], None, 16, 2, 64, 64),                                 # 16 blocks of rows for few keys: the streaming kernel
])
def test_importance_rows_in_lds(lens, prefix, hq, hkv, d, window):
    """Every launch shape of the importance kernel that holds the window rows in LDS, and the shapes next to
    its limits, against the oracle; the same bits on a second run."""
    chunked = prefix is not None
    klens = [a + b for a, b in zip(lens, prefix)] if chunked else None
    wl = W.make_custom("t", lens, klens, hq, hkv, d, 0 if chunked else window, "1/4", seed=91, chunked=chunked)
    dev = DeviceWorkload(wl)
    got = []
    for _ in range(2):
        dev.poison()
        dev.attn(True)
        torch.cuda.synchronize()
        got.append(dev.imp.clone())
    assert torch.equal(got[0], got[1])
    oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, window)
    rel_close(got[0].cpu().numpy().astype(np.float64), oI, "importance")


@pytest.mark.parametrize("lens,prefix,hq,hkv,d", [
    ([1, 37, 96, 8, 2], [5003, 9000, 4100, 31, 0], 16, 4, 128),             # 8 waves, 1 to 12 blocks
    ([130, 3, 71], [12001, 20000, 999], 16, 4, 128),                        # 16 waves
    ([0, 33, 290, 1], [700, 7000, 9777, 15000], 8, 8, 64),                  # head_dim 64, a sequence without rows
    ([5] * 31 + [40], [900 + 7 * i for i in range(32)], 12, 4, 64),         # G = 3, many sequences
])
def test_importance_of_uneven_chunks(lens, prefix, hq, hkv, d):
    """Chunks whose lengths differ and whose keys are more than the chip takes at once: every sequence gets
    groups of keys by its own number of rows.  The same sums as the streaming kernel up to the order of fp32
    additions (at most 1216 positive terms in a sum, 1e-4 relative), every key written."""
    klens = [a + b for a, b in zip(lens, prefix)]
    wl = W.make_custom("t", lens, klens, hq, hkv, d, 0, "1/4", seed=92, chunked=True)
    dev = DeviceWorkload(wl)
    got = []
    try:
        for keys in (0, 0, 128):
            pdd.set_option(pdd.OPT_IMPORTANCE_KEYS, keys)
            dev.poison()
            dev.attn(True)
            torch.cuda.synchronize()
            got.append(dev.imp.clone())
    finally:
        pdd.set_option(pdd.OPT_IMPORTANCE_KEYS, 0)
    assert torch.equal(got[0], got[1])
    rel_close(got[0].cpu().numpy().astype(np.float64), got[2].cpu().numpy().astype(np.float64), "importance")
    rel_close(got[0].cpu().numpy().astype(np.float64), oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, -1), "against the oracle")


def test_importance_of_a_very_large_group():
    """39676 query heads on one KV head: a (token, head) row number times the group's size passes 2^32, and the
    divided walks over the rows begin in the last heads of a token."""
    wl = W.make_custom("t", [9], [136], 39676, 1, 64, 0, "1/4", seed=93, gain=1.5, chunked=True)
    dev = DeviceWorkload(wl)
    desc, keep = pdd.make_desc(dev.q, dev.k, None, None, dev.cu_q, dev.cu_k, 9, 136, wl.scale, -1)
    nbytes = pdd.workspace_bytes(desc, pdd.CALL_TOKEN_IMPORTANCE)
    assert nbytes >= 2 * 136 * 4, "the rows are divided"
    dev.imp.fill_(float("nan"))
    lse = torch.from_numpy(oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale)[1]).float().cuda()
    pdd.token_importance(dev.q, dev.k, lse, dev.imp, dev.cu_q, dev.cu_k, 9, 136, wl.scale, -1,
                         workspace=torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
    oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, -1)
    rel_close(dev.imp.cpu().numpy().astype(np.float64), oI, "importance")
    del keep


@pytest.mark.parametrize("lens,klens,hq,hkv,planes", [
    ([130, 1, 1, 1, 1], [130, 1, 32, 301, 2501], 32, 8, 1),      # divided for its uneven lengths alone
    ([3, 1, 3, 1, 130], [3, 32, 303, 2501, 130], 16, 4, 3),      # by three if all were as long as the longest; by four as they are
])
def test_importance_scratch_too_small_or_misaligned(lens, klens, hq, hkv, planes):
    """Scratch that holds what lengths all alike would take is used, or refused if it is misaligned; scratch that only
    the uneven lengths make use of is not refused."""
    wl = W.make_custom("t", lens, klens, hq, hkv, 128, 0, "1/4", seed=94, chunked=True)
    dev = DeviceWorkload(wl)
    dev.attn(False)
    desc, keep = pdd.make_desc(dev.q, dev.k, None, None, dev.cu_q, dev.cu_k, dev.max_q, dev.max_k, wl.scale, -1)
    need, plane = pdd.workspace_bytes(desc, pdd.CALL_TOKEN_IMPORTANCE), hkv * wl.total_k * 4
    assert need == 4 * plane
    buf = torch.empty(need + 16, dtype=torch.uint8, device="cuda")

    def run(scratch):
        dev.imp.fill_(float("nan"))
        buf.fill_(0xFF)
        pdd.token_importance(dev.q, dev.k, dev.lse, dev.imp, dev.cu_q, dev.cu_k, dev.max_q, dev.max_k, wl.scale, -1,
                             workspace=scratch)
        torch.cuda.synchronize()
        return dev.imp.clone(), bool((buf != 0xFF).any())

    whole, _ = run(None)
    oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, -1)
    for size, used in ((need, True), (need - 1, planes > 1), (planes * plane, planes > 1), (planes * plane - 1, False)):
        got, wrote = run(buf[:size])
        assert wrote == used, size
        assert torch.equal(got, whole) or used
        rel_close(got.cpu().numpy().astype(np.float64), oI, f"importance, {size} bytes")
        if planes > 1 and size >= planes * plane:
            with pytest.raises(pdd.PddError, match="aligned"):
                run(buf[8:8 + size])
        else:
            got, wrote = run(buf[8:8 + size])
            assert torch.equal(got, whole) and not wrote
    del keep


def test_importance_key_widths_give_the_same_bits():
    """The importance kernel with 256 and with 128 keys per workgroup (the library picks by launch
    size): the same column sums bit for bit, on ragged prefill (windows that end inside a key
    slice, sequences shorter than a slice) and on chunks behind a prefix without scratch; the
    first against the oracle as well."""
    cases = [W.make_custom("t", [700, 33, 1290, 128, 5], None, 8, 2, 128, 96, "1/2", seed=71),
             W.make_custom("t", [300, 64], None, 6, 3, 64, 40, "1/2", seed=72),
             W.make_custom("t", [256, 77], [256 + 1500, 77 + 900], 8, 2, 128, 0, "1/4", seed=73, chunked=True)]
    try:
        for n, wl in enumerate(cases):
            dev = DeviceWorkload(wl)
            got = {}
            for keys in (256, 128):
                pdd.set_option(pdd.OPT_IMPORTANCE_KEYS, keys)
                dev.poison()
                dev.attn(True, use_workspace=False)
                torch.cuda.synchronize()
                got[keys] = dev.imp.clone()
            assert torch.equal(got[256], got[128]), f"case {n}"
            if n == 0:
                oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, wl.window)
                rel_close(got[128].cpu().numpy().astype(np.float64), oI, "128 keys per workgroup")
    finally:
        pdd.set_option(pdd.OPT_IMPORTANCE_KEYS, 0)


@pytest.mark.parametrize("name", ["c5", "c3", "c4"])
def test_results_are_bit_identical_run_to_run(name):
    """The whole path twice on the same inputs: identical bits.  Large launches matter here:
    a read of an MFMA result before its last pass had been written (an assembly instruction
    the compiler could not guard) once made the running max, and so the rounding of O and lse,
    depend on how the two waves of a SIMD interleaved."""
    wl = W.make_workload(name)
    dev = DeviceWorkload(wl)
    dev.step()
    torch.cuda.synchronize()
    ref = [x.copy() for x in dev.results()]
    for _ in range(1 if name == "c4" else 3):
        dev.poison()
        dev.step()
        torch.cuda.synchronize()
        for what, a, b in zip(("O", "lse", "importance", "indices", "mask"), ref, dev.results()):
            assert np.array_equal(a, b), f"{name}: {what} differs between two runs"


# ------------------------------------------------------------- selection alone
def _select_case(scores64, lens, ks, cand=None, rel_tie=1e-6):
    """Gate A: the oracle's scores rounded to fp32 go through the GPU select."""
    wl = W.make_custom("t", lens, None, 1, 1, 64, 0, seed=0)   # only cu_seqlens etc. are used
    wl.n_kv_heads = scores64.shape[0]
    wl.k_keep = np.array(ks, dtype=np.int32)
    if cand is not None:
        wl.cand_begin = np.array(cand[0], dtype=np.int32)
        wl.cand_end = np.array(cand[1], dtype=np.int32)
    dev = DeviceWorkload(wl)
    dev.poison()
    s32 = torch.from_numpy(scores64.astype(np.float32)).cuda()
    dev.select(scores=s32)
    torch.cuda.synchronize()
    idx, mask = dev.idx.cpu().numpy(), dev.mask.cpu().numpy()
    # exactness on what the kernel saw (fp32), tie allowance on the fp64 scores
    check_selection(scores64.astype(np.float32).astype(np.float64), idx, mask, wl, -1, "select fp32")
    check_selection(scores64, idx, mask, wl, rel_tie, "select fp64")
    return idx, mask


def test_select_ties_negative_values_and_ranges():
    rng = np.random.default_rng(5)
    lens = [1000, 1, 64, 4097]
    tot = sum(lens)
    s = rng.integers(0, 50, size=(3, tot)).astype(np.float64) / 8.0       # many exact ties
    s[1] = rng.standard_normal(tot)                                          # negatives
    s[2, :] = 0.25                                                           # all equal
    s[1, 5] = -0.0
    _select_case(s, lens, [300, 1, 10, 2048])
    _select_case(s, lens, [0, 0, 64, 4097])                                  # nothing / everything
    _select_case(s, lens, [100, 1, 5, 1000], cand=([10, 0, 32, 4], [900, 1, 40, 4000]))
    idx, _ = _select_case(s[2:3], lens, [7, 1, 3, 11])
    assert idx[0, :7].tolist() == list(range(7))                             # lowest indices win


def test_select_long_rows_beyond_lds_staging():
    rng = np.random.default_rng(6)
    lens = [40000, 33000]
    s = np.abs(rng.standard_normal((2, sum(lens)))) ** 3
    s[1, ::3] = s[1, 0]
    _select_case(s, lens, [4000, 16500])
    _select_case(s, lens, [1, 33000])


@pytest.mark.parametrize("n", [128, 129, 132, 4095, 4096, 4097, 8192, 16384, 32767])
def test_select_threshold_search_off_its_good_path(n):
    """Rows whose sample says nothing about them (every fourth score high, the position within a quad
    that is sampled; the rest of the keys in another range), two values, neighbouring floats, a few values far
    apart, a heavy tie among spread scores: k from 1 to n.  Exact."""
    rng = np.random.default_rng(n)
    x = np.arange(n)
    u = rng.random(n)
    rows = np.stack([np.where(x % 4 == 0, 1e6 + x, u), np.where(x % 4 == 0, u * 1e-6, 1.0 + u), np.where(u < 0.3, 2.0, -1.0),
                     1.0 + rng.integers(0, n, n) * 2.0 ** -23, 10.0 ** rng.integers(-30, 30, n),
                     np.where(u < 0.5, 0.7, rng.random(n) ** 6)]).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    cu = np.array([0, n], dtype=np.int32)
    scores = dev(rows)
    for k in sorted({1, 2, n // 10, n // 4, n // 2, 3 * n // 4, n - 1, n}):
        keep = np.array([k], dtype=np.int32)
        idx = torch.full((len(rows), k), -7, dtype=torch.int32, device="cuda")
        mask = torch.full(rows.shape, 9, dtype=torch.uint8, device="cuda")
        pdd.select_topk(scores, dev(cu), n, dev(keep), dev(np.array([0, k], dtype=np.int32)), k, idx, mask, None, None, cu)
        want_idx, want_mask = oracle.select_topk(rows.astype(np.float64), cu, keep)
        assert np.array_equal(idx.cpu().numpy(), want_idx), f"k = {k}"
        assert np.array_equal(mask.cpu().numpy(), want_mask), f"k = {k}"


@pytest.mark.parametrize("n", [300, 4096, 4097, 8192, 20606, 32768])
def test_select_runs_of_equal_scores(n):
    """More equal scores than the last step of the search ranks: five values, most of them zero, 24 neighbouring values at
    doubling distances, the same beside one score far off.  As tokens and, up
    to 8192, as sentences of one token.  Exact."""
    rng = np.random.default_rng(n)
    u = rng.random(n)
    near = (np.uint32(0x3F000000) + (np.uint32(1) << rng.integers(0, 24, n).astype(np.uint32))).view(np.float32)
    far = near.copy()
    far[n // 3] = 1e30
    rows = np.stack([rng.integers(0, 5, n), np.where(u < 0.9, 0.0, u), near, far]).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    cu = np.array([0, n], dtype=np.int32)
    scores = dev(rows)
    for k in sorted({1, 2, n // 20, n // 4, n // 2, 3 * n // 4, n - 1, n}):
        keep = np.array([k], dtype=np.int32)
        idx = torch.full((len(rows), k), -7, dtype=torch.int32, device="cuda")
        mask = torch.full(rows.shape, 9, dtype=torch.uint8, device="cuda")
        pdd.select_topk(scores, dev(cu), n, dev(keep), dev(np.array([0, k], dtype=np.int32)), k, idx, mask, None, None, cu)
        want_idx, want_mask = oracle.select_topk(rows.astype(np.float64), cu, keep)
        assert np.array_equal(idx.cpu().numpy(), want_idx), f"k = {k}"
        assert np.array_equal(mask.cpu().numpy(), want_mask), f"k = {k}"
        if n <= 8192:
            sent = torch.full(rows.shape, 9, dtype=torch.uint8, device="cuda")
            pdd.select_sentences(scores, dev(cu), n, dev(cu), dev(np.arange(1, n + 1, dtype=np.int32)), n, dev(keep), pdd.SENT_SUM,
                                 None, None, sent, None, None, cu)
            assert np.array_equal(sent.cpu().numpy(), want_mask), f"sentences, k = {k}"


@pytest.mark.parametrize("n,pool", [(4097, 0), (6001, 0), (8192, 2), (16384, 0), (20606, 2), (32768, 0)])
def test_select_long_rows_of_two_and_three_scores(n, pool):
    """Two scores, alone and with a rare one between, above or below, kept to one less than the higher ones, to all of
    them and to one more, to the rare ones and past them.  With and without pooling by the maximum; exact."""
    rng = np.random.default_rng(n)
    at, rare = rng.random(n), rng.random(n) < 0.01
    row = lambda low, high, other: np.where(rare, other, np.where(at < (0.05 if pool else 0.45), high, low))
    rows = np.stack([row(-2, 3, 3), row(-2, 3, 0.5), row(-2, 3, 7), row(-2, 3, -5), row(0, 1e-45, 0)]).astype(np.float32)
    ranked = oracle.pool_scores(rows.astype(np.float64), np.array([0, n]), 2 * pool + 1, "max") if pool else rows
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    cu = np.array([0, n], dtype=np.int32)
    counts = {int((r >= v).sum()) for r in ranked for v in np.unique(r)}
    for k in sorted({min(max(c + d, 1), n) for c in counts for d in (-1, 0, 1)}):
        keep = np.array([k], dtype=np.int32)
        idx = torch.full((len(rows), k), -7, dtype=torch.int32, device="cuda")
        mask = torch.full(rows.shape, 9, dtype=torch.uint8, device="cuda")
        args = (dev(rows), dev(cu), n, dev(keep), dev(np.array([0, k], dtype=np.int32)), k, idx, mask)
        if pool:
            pdd.select_topk_pooled(*args, 2 * pool + 1, pdd.POOL_MAX, None, None, None, cu)
        else:
            pdd.select_topk(*args, None, None, cu)
        want_idx, want_mask = oracle.select_topk(ranked, cu, keep)
        assert np.array_equal(idx.cpu().numpy(), want_idx), f"k = {k}"
        assert np.array_equal(mask.cpu().numpy(), want_mask), f"k = {k}"


@pytest.mark.parametrize("n", [5, 128, 300, 4097, 32768])
def test_select_key_of_the_lowest_nan(n):
    """A score whose bits are all ones (a buffer filled with 0xFF bytes) ranks below every other value
    and is still a candidate: it takes its slot when everything is kept, and none before."""
    rng = np.random.default_rng(n)
    bits = rng.standard_normal((2, n)).astype(np.float32).view(np.uint32)
    low = rng.random((2, n)) < 0.4
    low[:, :2], bits[1, -1] = (True, False), np.uint32(0xFF800000)            # -infinity
    low[1, -1] = False
    bits[low] = 0xFFFFFFFF
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    cu, scores = np.array([0, n], dtype=np.int32), dev(bits.view(np.float32))
    rank = np.where(low, -np.inf, np.maximum(bits.view(np.float32), np.float32(-1e30))).astype(np.float64)
    for k in sorted({1, n - int(low.sum(1).max()), n - 1, n}):
        idx = torch.full((2, k), -7, dtype=torch.int32, device="cuda")
        mask = torch.full((2, n), 9, dtype=torch.uint8, device="cuda")
        keep = np.array([k], dtype=np.int32)
        pdd.select_topk(scores, dev(cu), n, dev(keep), dev(np.array([0, k], dtype=np.int32)), k, idx, mask, None, None, cu)
        want_idx, want_mask = oracle.select_topk(rank, cu, keep)
        assert np.array_equal(idx.cpu().numpy(), want_idx) and np.array_equal(mask.cpu().numpy(), want_mask), f"k = {k}"


@pytest.mark.parametrize("dist", ["spread", "equal", "low_bits", "signs", "infinities"])
@pytest.mark.parametrize("lens", [[32769], [36864, 5, 0, 4097, 4096], [131071, 40000]])
def test_select_rows_divided_over_workgroups(lens, dist):
    """Rows of more than 32768 candidates with a workspace: chunks of 4096 that end on a remainder, sequences
    shorter than a chunk and empty ones, candidate ranges, k = 0 and k beyond the candidates, at odd
    addresses; scores that differ only in their last digit, ties across chunks.  Exact."""
    rng = np.random.default_rng(sum(lens))
    heads, cu = 2, np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    shape = (heads, sum(lens))
    scores = {"spread": rng.random(shape) ** 6, "equal": np.full(shape, 0.25), "signs": rng.normal(size=shape),
              "low_bits": np.float32(1.0) + rng.integers(0, 900, shape) * 2.0 ** -23,
              "infinities": np.where(rng.random(shape) < 0.6, -np.inf, rng.choice([np.inf, 1.0, -0.0, 0.0], shape))}
    s32 = scores[dist].astype(np.float32)
    n = np.array(lens, dtype=np.int32)
    for begin, end, k in ((n * 0, n, n // 3), (n // 7, n - n // 9, n // 2), (n // 7, n - n // 9, n * 0), (n // 2, n, n)):
        cand_b, cand_e = begin.astype(np.int32), end.astype(np.int32)
        k_keep = np.minimum(k, n).astype(np.int32)
        cu_keep = np.concatenate([[0], np.cumsum(k_keep)]).astype(np.int32)
        desc = pdd.AttnDesc()
        desc.batch, desc.n_q_heads, desc.n_kv_heads, desc.head_dim = len(lens), heads, heads, 128
        desc.total_q = desc.total_k = int(cu[-1])
        desc.max_seqlen_q = desc.max_seqlen_k = max(lens)
        need = pdd.workspace_bytes(desc, pdd.CALL_SELECT_TOPK)
        assert need > 0
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
        sc = torch.from_numpy(np.concatenate([[9.0], s32.ravel()]).astype(np.float32)).cuda()[1:].view(shape)   # 4-byte aligned
        idx = torch.full((heads, int(cu_keep[-1])), -7, dtype=torch.int32, device="cuda")
        mask = torch.full((s32.size + 3,), 9, dtype=torch.uint8, device="cuda")[3:].view(shape)
        dev = lambda a: torch.from_numpy(a).cuda()
        pdd.select_topk(sc, dev(cu), max(lens), dev(k_keep), dev(cu_keep), int(cu_keep[-1]), idx, mask, dev(cand_b),
                        dev(cand_e), cu, workspace=ws)
        taken = np.minimum(k_keep, cand_e - cand_b)
        want_idx, want_mask = oracle.select_topk(s32.astype(np.float64), cu, taken, cand_b, cand_e)
        got, cu_want = idx.cpu().numpy(), np.concatenate([[0], np.cumsum(taken)])
        for b in range(len(lens)):
            row = got[:, cu_keep[b]:cu_keep[b + 1]]
            assert np.array_equal(row[:, :taken[b]], want_idx[:, cu_want[b]:cu_want[b + 1]])
            assert (row[:, taken[b]:] == -1).all()
        assert np.array_equal(mask.cpu().numpy(), want_mask)
        assert (ws != 0xFF).any() or not taken.any(), "the scratch was not used"


def _sample_of_divided_row(n):
    """Where a divided row of n candidates is sampled: one place in each of 1024 equal pieces."""
    i = np.arange(1024, dtype=np.uint64)
    mix = (i * np.uint64(2654435761)) & np.uint64(0xffffffff)
    return (((i << np.uint64(16)) | (mix >> np.uint64(16))) * np.uint64(n) >> np.uint64(26)).astype(np.int64)


@pytest.mark.parametrize("heads,n,kind", [
    (1, 40000, "spread"), (40, 40000, "spread"), (64, 40000, "spread"),      # 4096, 8192 and 16384 candidates to a workgroup
    (1, 300000, "spread"), (3, 1100000, "few"),                              # more than 64 and than 32 workgroups to a row
    (2, 70000, "octaves"),                                                   # bins wider than 16 bits
    (1, 70000, "sample above"), (1, 70000, "sample below"),                  # the sample says nothing of the row
    (1, 300000, "one bin")])                                                 # more keys in the threshold's bin than are listed
def test_select_divided_rows_off_the_good_path(heads, n, kind):
    rng = np.random.default_rng(n)
    s = rng.random((heads, n)) ** 6
    k = n // 10
    if kind == "few":
        s = rng.integers(0, 5, (heads, n)).astype(np.float64)
    elif kind == "octaves":
        s, k = np.exp(20 * rng.normal(size=(heads, n))), 40
    elif kind == "sample above":
        s[:, _sample_of_divided_row(n)] += 2.0
    elif kind == "sample below":
        s[:, _sample_of_divided_row(n)] -= 2.0
    elif kind == "one bin":
        s, k = np.where(rng.random((heads, n)) < 0.5, 1.0 + rng.random((heads, n)) * 1e-4, rng.random((heads, n))), n // 2
    s32 = s.astype(np.float32)
    cu, k_keep = np.array([0, n], dtype=np.int32), np.array([k], dtype=np.int32)
    desc = pdd.AttnDesc()
    desc.batch, desc.n_kv_heads, desc.max_seqlen_k = 1, heads, n
    need = pdd.workspace_bytes(desc, pdd.CALL_SELECT_TOPK)
    assert need > 0
    guard = 4096
    ws = torch.full((need + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    dev = lambda a: torch.from_numpy(a).cuda()
    idx = torch.full((heads, k), -7, dtype=torch.int32, device="cuda")
    mask = torch.full((heads, n), 9, dtype=torch.uint8, device="cuda")
    pdd.select_topk(dev(s32), dev(cu), n, dev(k_keep), dev(np.array([0, k], dtype=np.int32)), k, idx, mask, None, None, cu,
                    workspace=ws[:need])
    assert (ws[need:] == 0xA5).all(), "written past the scratch"
    got, m = idx.cpu().numpy(), mask.cpu().numpy()
    for h in range(heads):
        want = np.sort(np.argsort(-s32[h], kind="stable")[:k])           # ties: the lower index
        assert np.array_equal(got[h], want)
        assert np.array_equal(np.flatnonzero(m[h]), want)


@pytest.mark.parametrize("heads,n,values", [
    (8, 131072, 7), (40, 40000, 7), (1, 600000, 7),          # the threshold's value is neither edge: 18700, 5700 and 86000 keys of a bin
    (2, 400000, "pair"),                                     # two neighbouring values, 40000 keys of a bin that are not one value
    (1, 900000, "pair, few bits"), (1, 300000, "octaves"),   # bins of one value each; the outermost bins, of many
])
@pytest.mark.parametrize("at", [0.5, 0.47])
def test_select_divided_rows_with_more_keys_in_a_bin_than_lds_holds(heads, n, values, at):
    """Rows of few values, or of two common ones among many, kept to about the middle: the threshold's bin holds more
    keys than a workgroup lists in LDS (or, in the shortest row, many)."""
    rng = np.random.default_rng(n)
    u = rng.random((heads, n))
    if values == 7:
        s = np.floor(7 * u) / 7 + 0.1
    elif values == "octaves":
        s = np.where(u < 0.4, 1.0 + u, np.where(u < 0.6, np.exp2(np.floor(200 * rng.random((heads, n)) - 100)), -1.0 - u))
        s[u < 0.4] += 2.0 ** 101
    else:
        a = np.float32(0.55)
        b = np.nextafter(a, np.float32(1))
        s = np.where(u < 0.45, 0.5 * u, np.where(u < 0.5, a, np.where(u < 0.55, b, 0.6 + (u - 0.55) * (1e3 if values == "pair" else 1e-3))))
    s32 = s.astype(np.float32)
    k = int(at * n)
    cu, k_keep = np.array([0, n], dtype=np.int32), np.array([k], dtype=np.int32)
    desc = pdd.AttnDesc()
    desc.batch, desc.n_kv_heads, desc.max_seqlen_k = 1, heads, n
    need = pdd.workspace_bytes(desc, pdd.CALL_SELECT_TOPK)
    assert need > 0
    ws = torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda")
    dev = lambda a: torch.from_numpy(a).cuda()
    idx = torch.full((heads, k), -7, dtype=torch.int32, device="cuda")
    mask = torch.full((heads, n), 9, dtype=torch.uint8, device="cuda")
    pdd.select_topk(dev(s32), dev(cu), n, dev(k_keep), dev(np.array([0, k], dtype=np.int32)), k, idx, mask, None, None, cu, workspace=ws)
    got, m = idx.cpu().numpy(), mask.cpu().numpy()
    for h in range(heads):
        want = np.sort(np.argsort(-s32[h], kind="stable")[:k])           # ties: the lower index
        assert np.array_equal(got[h], want)
        assert np.array_equal(np.flatnonzero(m[h]), want)


@pytest.mark.parametrize("name", ["c1", "c2", "c3", "c5", "c4"])
def test_gate_a_oracle_scores_of_every_configuration(name):
    """The oracle's importance of each benchmark configuration, rounded to fp32, through the GPU
    selection with that configuration's own candidate ranges and k: the set must be the
    oracle's, except inside the 1e-6 relative tie band.  The row lengths 512 / 4096, 7898,
    8448 and 32768 take the register-resident kernel with 4, 8, 16 and 32 keys per thread."""
    wl = W.make_workload(name)
    window = -1 if wl.chunked else wl.window
    oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, window)
    dev = DeviceWorkload(wl)
    dev.poison()
    s32 = oI.astype(np.float32)
    dev.select(scores=torch.from_numpy(s32).cuda())
    torch.cuda.synchronize()
    idx, mask = dev.idx.cpu().numpy(), dev.mask.cpu().numpy()
    check_selection(s32.astype(np.float64), idx, mask, wl, -1, f"{name} gate A fp32")
    swapped = check_selection(oI, idx, mask, wl, 1e-6, f"{name} gate A fp64")
    print(f"{name}: gate A swapped inside the tie band: {swapped}")


@pytest.mark.parametrize("n", [3000, 4096, 8000, 16384, 20000, 32768])
def test_select_exact_in_every_register_variant(n):
    """Exact selection (ties, candidate ranges, k = 0 / everything) at row lengths that take the
    register-resident kernel with 4, 8, 16 and 32 keys per thread."""
    rng = np.random.default_rng(n)
    lens = [n, 1, n // 3]
    tot = sum(lens)
    s = rng.integers(0, 200, size=(3, tot)).astype(np.float64) / 16.0      # many exact ties
    s[1] = rng.standard_normal(tot) ** 3
    s[2, : n // 2] = 0.125                                                   # a long plateau
    _select_case(s, lens, [n // 10, 1, n // 6])
    _select_case(s, lens, [n, 0, 1])
    _select_case(s, lens, [n // 4, 1, 5], cand=([7, 0, 1], [n - 5, 1, n // 3 - 1]))


@pytest.mark.parametrize("kind", ["above", "below", "equal", "one bin", "one bin, many"])
@pytest.mark.parametrize("n", [4097, 8193, 20606, 32767, 32768])
def test_select_register_rows_that_their_sample_misjudges(n, kind):
    """Rows of 4097 to 32768 keys bracket the threshold by 1024 of their scores.  Here those say nothing about
    the others: all above or below them, all equal, or in one bin of the histogram with many keys that differ."""
    rng = np.random.default_rng(n)
    tid = np.arange(1024)
    at = (tid // 2) * n // 512 + 4 * (tid % 2)
    s = rng.random((3, n))
    if kind == "above":
        s[:, at] += 2.0
    elif kind == "below":
        s[:, at] -= 2.0
    elif kind == "equal":
        s[:, at] = 0.5
    elif kind == "one bin":
        s = 1.0 + s * 1e-4
        s[:, at[::7]] = 1e30
    else:
        s = np.where(rng.random((3, n)) < 0.5, 1.0 + s * 1e-4, s)
    s = s.astype(np.float32).astype(np.float64)
    for k in (1, 2, n // 100, n // 4, n // 2, n - 1, n):
        _select_case(s, [n], [k], rel_tie=-1)


def _score_row(rng, kind, n):
    """Score distributions that stress the threshold search: its probes interpolate on the key value."""
    if kind == 0:
        return rng.standard_normal(n)
    if kind == 1:
        return np.exp(rng.standard_normal(n) * 3 - 9)                             # heavy tail
    if kind == 2:
        return rng.integers(0, 7, n).astype(np.float64) / 4                       # few distinct values
    if kind == 3:
        return np.full(n, 0.375)                                                  # constant
    if kind == 4:
        return rng.standard_normal(n) * 10.0 ** rng.integers(-30, 30, n)          # 60 decades, both signs
    if kind == 5:
        x = np.sort(rng.random(n))
        return x if rng.random() < .5 else x[::-1].copy()                         # sorted either way
    if kind == 6:
        x = rng.random(n) ** 8
        x[rng.integers(0, n, max(1, n // 50))] = 1e30                             # far outliers
        return x
    x = np.zeros(n)
    x[rng.integers(0, n, max(1, n // 100))] = rng.random(max(1, n // 100))       # mostly zero
    return x


@pytest.mark.parametrize("seed", range(4))
def test_select_random_distributions_exact(seed):
    """Seeded random rows of eight kinds (see _score_row), random lengths up to every register
    size, candidate ranges, keep counts (0 and everything included) and tensor offsets: the
    selection on the fp32 scores is exactly the oracle's."""
    rng = np.random.default_rng(900 + seed)
    for it in range(12):
        B, H = int(rng.integers(1, 4)), int(rng.integers(1, 3))
        cap = [700, 4096, 5000, 8192, 12000, 16384, 20000, 32768][int(rng.integers(0, 8))]
        lens = [int(rng.integers(1, cap + 1)) for _ in range(B)]
        lens[int(rng.integers(0, B))] = cap
        s = np.stack([np.concatenate([_score_row(rng, int(rng.integers(0, 8)), n) for n in lens]) for _ in range(H)])
        s = s.astype(np.float32).astype(np.float64)
        cb = [int(rng.integers(0, max(1, n // 3))) if rng.random() < .5 else 0 for n in lens]
        ce = [int(rng.integers(b, n + 1)) if rng.random() < .5 else n for b, n in zip(cb, lens)]
        ks = [int(rng.integers(0, e - b + 1)) if rng.random() < .8 else (e - b) for b, e in zip(cb, ce)]
        wl = W.make_custom("t", lens, None, 1, 1, 64, 0, seed=0)
        wl.n_kv_heads = H
        wl.k_keep = np.array(ks, dtype=np.int32)
        wl.cand_begin, wl.cand_end = np.array(cb, dtype=np.int32), np.array(ce, dtype=np.int32)
        dev = DeviceWorkload(wl)
        dev.poison()
        off = int(rng.integers(0, 4))
        flat = torch.zeros(H * sum(lens) + 4, dtype=torch.float32, device="cuda")
        view = flat[off:off + H * sum(lens)].view(H, sum(lens))
        view.copy_(torch.from_numpy(s.astype(np.float32)))
        dev.select(scores=view)
        torch.cuda.synchronize()
        check_selection(s, dev.idx.cpu().numpy(), dev.mask.cpu().numpy(), wl, -1,
                        f"seed {seed} case {it}: lens={lens} keep={ks} cand={cb}..{ce} offset={off}")


@pytest.mark.parametrize("n", [1000, 6000, 12000, 32768])
@pytest.mark.parametrize("score_off,mask_off", [(1, 0), (0, 1), (3, 2)])
def test_select_unaligned_tensors(n, score_off, mask_off):
    """Score and mask tensors that do not start on a 16-byte / 4-byte boundary: the kernel takes the
    candidates before the first 16-byte boundary of a row one by one and writes the mask bytes
    singly where its quads do not line up with 4-byte words (1, 2, 4, 8 quads per thread at these
    lengths); same exactness."""
    rng = np.random.default_rng(n + 1)
    lens = [n, 77]
    heads = 2
    s = rng.integers(0, 300, size=(heads, sum(lens))).astype(np.float64) / 32.0
    s[1] = rng.standard_normal(sum(lens))
    wl = W.make_custom("t", lens, None, 1, 1, 64, 0, seed=0)
    wl.n_kv_heads = heads
    wl.k_keep = np.array([n // 7, 30], dtype=np.int32)
    dev = DeviceWorkload(wl)
    dev.poison()
    flat = torch.zeros(heads * sum(lens) + 4, dtype=torch.float32, device="cuda")
    view = flat[score_off:score_off + heads * sum(lens)].view(heads, sum(lens))
    view.copy_(torch.from_numpy(s.astype(np.float32)))
    assert view.data_ptr() % 16 == 4 * score_off
    mflat = torch.full((heads * sum(lens) + 4,), 9, dtype=torch.uint8, device="cuda")
    dev.mask = mflat[mask_off:mask_off + heads * sum(lens)].view(heads, sum(lens))
    assert dev.mask.data_ptr() % 4 == mask_off
    dev.select(scores=view)
    torch.cuda.synchronize()
    idx, mask = dev.idx.cpu().numpy(), dev.mask.cpu().numpy()
    check_selection(s.astype(np.float32).astype(np.float64), idx, mask, wl, -1, "unaligned fp32")
    guard = mflat.cpu().numpy()                     # nothing written outside the mask view
    assert (guard[:mask_off] == 9).all() and (guard[mask_off + heads * sum(lens):] == 9).all()


# ------------------------------------------------------ benchmark configurations
def test_c2_llama_layer_full():
    wl = W.make_workload("c2")
    o_err, swapped = run_and_compare(wl)
    print(f"c2: O err {o_err:.4f}, swapped {swapped}")
    assert swapped == 0


def _sample_rows(wl, per_seq_random, tile=256, seed=0, first=64):
    """Window rows, the first `first` rows, every `tile`-row boundary +- 1 and seeded random rows."""
    rng = np.random.default_rng(seed)
    rows = []
    for b in range(wl.batch):
        qs, nq = int(wl.cu_seqlens_q[b]), int(wl.seqlens_q[b])
        w = nq if wl.chunked else min(wl.window, nq)
        loc = set(range(nq - w, nq)) | set(range(min(nq, first)))
        for t in range(tile, nq, tile):
            loc |= {t - 1, t, t + 1} & set(range(nq))
        loc |= set(int(x) for x in rng.integers(0, nq, size=per_seq_random))
        rows += [qs + i for i in sorted(loc)]
    return np.array(rows, dtype=np.int32)


@pytest.mark.parametrize("waves", [4, 8])
def test_head_dim_64_longer_prompts_sampled_rows(waves):
    """The head_dim-64 kernel on prompts of many tiles (the graded configurations with d = 64
    stop at 512 tokens)."""
    wl = W.make_custom("t", [3000, 1111], None, 8, 2, 64, 64, "1/4", seed=77)
    o_err, swapped = run_and_compare(wl, rows=_sample_rows(wl, 48), waves=waves, label=f"d64 long w={waves}")
    assert swapped == 0


# On 256 compute units: 4 waves, two workgroups to a unit, and 8 waves (576 and 448 tiles of 256 rows); 64 queries to a wave; 4 waves,
# three to a unit (all tiles take the chip as long as the longest walk takes one)
@pytest.mark.parametrize("lens,form", [([700, 1, 513], pdd.ATTN_4_WAVES), ([1700], pdd.ATTN_8_WAVES), ([1700, 1, 1690], pdd.ATTN_WIDE),
                                       ([2100], pdd.ATTN_4_WAVES)])
def test_head_dim_64_workgroup_choice_gives_the_same_bits(lens, form):
    wl = W.make_custom("t", lens, None, 64, 8, 64, 32, "1/4", seed=21)
    assert DeviceWorkload(wl).attn_form() == form
    runs = []
    for waves in (0, 4, 8):
        dev = DeviceWorkload(wl)
        dev.poison()
        pdd.set_option(pdd.OPT_ATTN_WAVES, waves)
        try:
            dev.step()
            runs.append(dev.results())
        finally:
            pdd.set_option(pdd.OPT_ATTN_WAVES, 0)
    for other in runs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(runs[0], other))
    rows = np.array([0, 1, 127, 128, 255, 256, len(wl.q) - 1])
    oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, rows=rows)
    assert np.abs(runs[0][0][rows] - oO).max() <= O_ATOL
    rel_close(runs[0][1][:, rows], oL, "lse")


def test_c3_ragged_batch_sampled_rows():
    wl = W.make_workload("c3")
    rows = _sample_rows(wl, 48)
    o_err, swapped = run_and_compare(wl, rows=rows)
    print(f"c3: {len(rows)} rows, O err {o_err:.4f}, swapped {swapped}")
    assert swapped == 0


def test_c4_long_prompt_sampled_rows():
    """O and log-sum-exp on every window row, the first 256 rows, every 256-row workgroup
    boundary +- 1 and 2048 seeded random rows (all 32 heads each); importance and the
    selection in full."""
    wl = W.make_workload("c4")
    rows = _sample_rows(wl, 2048, tile=256, first=256)
    o_err, swapped = run_and_compare(wl, rows=rows)
    print(f"c4: {len(rows)} rows, O err {o_err:.4f}, swapped {swapped}")
    assert swapped == 0


def test_prompt_of_131072_tokens_sampled_rows():
    """The paper's prompts reach hundreds of thousands of tokens: one 131072-token prompt (2 query
    heads on 1 KV head) through the whole path: 512 query tiles, 2048 K/V tiles for the last of
    them, tile offsets beyond 2^25 bytes, the radix selection.  O and log-sum-exp on the window
    rows, the first rows, every 8192nd workgroup boundary +- 1 and 64 seeded random rows;
    importance and the selection in full."""
    wl = W.make_custom("t", [131072], None, 2, 1, 128, 128, "1/8", seed=131)
    rows = _sample_rows(wl, 64, tile=8192, first=64)
    o_err, swapped = run_and_compare(wl, rows=rows)
    print(f"131072 tokens: {len(rows)} rows, O err {o_err:.4f}, swapped {swapped}")
    assert swapped == 0


@pytest.mark.skipif(os.environ.get("PDD_FULL_C4") != "1",
                    reason="about 10 minutes of fp64 oracle time; set PDD_FULL_C4=1")
def test_c4_long_prompt_every_row():
    """Every row of the 32k-token configuration against the oracle, in chunks that print
    their progress."""
    wl = W.make_workload("c4")
    dev = DeviceWorkload(wl)
    dev.poison()
    dev.step()
    O, lse, imp, idx, mask = dev.results()
    worst_o, worst_l = 0.0, 0.0
    step = 1024
    for r0 in range(0, wl.total_q, step):
        rows = np.arange(r0, min(r0 + step, wl.total_q), dtype=np.int32)
        oO, oL = oracle.attention(wl.q, wl.k, wl.v, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, rows=rows)
        worst_o = max(worst_o, float(np.abs(O[rows] - oO).max()))
        rel = np.abs(lse[:, rows] - oL) / np.maximum(np.abs(oL), 1e-6)
        worst_l = max(worst_l, float(rel.max()))
        print(f"c4 full: rows {r0}..{rows[-1]}: O max-abs {worst_o:.4g}, lse rel {worst_l:.3g}", flush=True)
        assert worst_o <= O_ATOL and worst_l <= REL
    oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, wl.window)
    rel_close(imp, oI, "c4 full importance")
    swapped = check_selection(oI, idx, mask, wl, REL, "c4 full select")
    irel = float((np.abs(imp - oI) / np.maximum(np.abs(oI), 1e-6)).max())
    print(f"c4 full: O max-abs {worst_o:.4g}, lse rel {worst_l:.3g}, importance rel {irel:.3g}, "
          f"gate-B swaps {swapped}", flush=True)
    assert swapped == 0


def test_c4h_heavy_hitters_are_selected():
    """Boosted-query variant: the marked keys carry most of the window mass, so
    the selection must contain (nearly) all of them; importance and indices
    still match the oracle."""
    wl = W.make_workload("c4h", n_override=8192)
    dev = DeviceWorkload(wl)
    dev.step()
    _, swapped = compare_all(wl, dev, rows=_sample_rows(wl, 32), label="c4h")
    idx = dev.idx.cpu().numpy()
    heavy = wl.extra["heavy_positions"]
    for g in range(wl.n_kv_heads):
        frac = np.isin(heavy[g], idx[g]).mean()
        assert frac > 0.9, f"head {g}: only {frac:.2f} of heavy keys kept"


def test_c5_chunked_catch_up():
    wl = W.make_workload("c5")
    rows = _sample_rows(wl, 0)[::4]          # every 4th chunk row of each sequence
    o_err, swapped = run_and_compare(wl, rows=rows)
    print(f"c5: {len(rows)} rows, O err {o_err:.4f}, swapped {swapped}")
    assert swapped == 0


# ------------------------------------------------------------------- bit stream
def test_pack_mask_bit_exact():
    rng = np.random.default_rng(8)
    lens = [13, 64, 0, 1000, 7, 4096 + 3]
    rows = 3
    m = (rng.random((rows, sum(lens))) < 0.3).astype(np.uint8) * rng.integers(1, 255, size=(rows, sum(lens))).astype(np.uint8)
    want, cu_bytes = oracle.pack_mask(m, np.concatenate([[0], np.cumsum(lens)]))
    cu_k = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device="cuda")
    out = torch.full((rows, int(cu_bytes[-1])), 0xAA, dtype=torch.uint8, device="cuda")
    pdd.pack_mask(torch.from_numpy(m).cuda(), cu_k, max(lens), torch.from_numpy(cu_bytes).cuda(),
                  int(cu_bytes[-1]), out, np.concatenate([[0], np.cumsum(lens)]))
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want)
    # end to end: the mask produced by the selection kernel
    wl = W.make_custom("t", [300, 77], None, 4, 2, 128, 40, "3/10", seed=5)
    dev = DeviceWorkload(wl)
    dev.step()
    want, cu_bytes = oracle.pack_mask(dev.mask.cpu().numpy(), wl.cu_seqlens_k)
    out = torch.empty((wl.n_kv_heads, int(cu_bytes[-1])), dtype=torch.uint8, device="cuda")
    pdd.pack_mask(dev.mask, dev.cu_k, dev.max_k, torch.from_numpy(cu_bytes).cuda(), int(cu_bytes[-1]), out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want)
    assert int(np.unpackbits(out.cpu().numpy()[0]).sum()) == int(wl.k_keep.sum())


# ------------------------------------------------------------------ 1-D pooling
# Row lengths per case: the longest row decides the kernel for the whole launch, so each case
# stays inside one class: register-resident with 4 / 8 / 16 / 32 keys per thread (longest row
# <= 4096 / 8192 / 16384 / 32768), or the radix kernel for longer rows.
_POOL_CASES = {
    "reg4": ([700, 3, 1, 4096], [70, 2, 1, 1500], [10, 0, 0, 0], [690, 3, 1, 4096]),
    "reg8": ([700, 3, 1, 5000], [70, 2, 1, 1500], [10, 0, 0, 0], [690, 3, 1, 5000]),
    "reg16": ([12000, 1, 9000], [1200, 1, 4500], [0, 0, 100], [12000, 1, 8000]),
    "reg32": ([30000, 2, 17000], [3000, 1, 17000], [5, 0, 0], [29990, 2, 17000]),
    "radix": ([700, 3, 40000], [70, 2, 4000], [10, 0, 100], [690, 3, 39000]),
}


@pytest.mark.parametrize("mode,kernel", [("max", 5), ("avg", 7), ("avg", 1), ("max", 33)])
@pytest.mark.parametrize("case", list(_POOL_CASES))
def test_pooled_selection(case, mode, kernel):
    lens, keep, cb, ce = _POOL_CASES[case]
    rng = np.random.default_rng(11)
    heads = 2
    s32 = (rng.random((heads, sum(lens))) ** 6).astype(np.float32)
    s32[1, 100:140] = 0.5                           # a plateau: ties after max pooling
    wl = W.make_custom("t", lens, None, 1, 1, 64, 0, seed=0)
    wl.n_kv_heads = heads
    wl.k_keep = np.array(keep, dtype=np.int32)
    wl.cand_begin = np.array(cb, dtype=np.int32)
    wl.cand_end = np.array(ce, dtype=np.int32)
    want_pooled = oracle.pool_scores(s32.astype(np.float64), wl.cu_seqlens_k, kernel, mode)
    dev = DeviceWorkload(wl)
    dev.poison()
    pooled = torch.full((heads, sum(lens)), float("nan"), dtype=torch.float32, device="cuda")
    pdd.select_topk_pooled(torch.from_numpy(s32).cuda(), dev.cu_k, dev.max_k, dev.k_keep, dev.cu_keep,
                           dev.total_keep, dev.idx, dev.mask, kernel,
                           pdd.POOL_MAX if mode == "max" else pdd.POOL_AVG, pooled,
                           dev.cand_b, dev.cand_e, wl.cu_seqlens_k)
    torch.cuda.synchronize()
    got_pooled = pooled.cpu().numpy().astype(np.float64)
    if mode == "max":
        assert np.array_equal(got_pooled, want_pooled)            # exact: a maximum of fp32 values
    else:
        np.testing.assert_allclose(got_pooled, want_pooled, rtol=1e-6, atol=1e-12)
    # the selection is exact on the scores the kernel ranked, and matches the fp64 pooling up to ties
    check_selection(got_pooled, dev.idx.cpu().numpy(), dev.mask.cpu().numpy(), wl, -1, "pooled fp32")
    check_selection(want_pooled, dev.idx.cpu().numpy(), dev.mask.cpu().numpy(), wl, 1e-6, "pooled fp64")


@pytest.mark.parametrize("mode", ["max", "avg"])
@pytest.mark.parametrize("kernel", [3, 129, 1025])
@pytest.mark.parametrize("lens", [[1, 3, 4096, 300], [4097, 8193], [32768]])
def test_pooled_selection_windows(lens, kernel, mode):
    """Windows of the smallest and the largest size around the edges of a step of 4096 keys, wider than the
    sequence, and reaching keys outside the candidate range; negative scores.  Same checks as above."""
    rng = np.random.default_rng(kernel)
    wl = W.make_custom("t", lens, None, 1, 1, 64, 0, seed=0)
    wl.n_kv_heads = 2
    s32 = rng.normal(size=(2, sum(lens))).astype(np.float32)
    n = np.array(lens, dtype=np.int32)
    wl.cand_begin, wl.cand_end = n // 5, n - n // 6
    wl.k_keep = ((wl.cand_end - wl.cand_begin + 2) // 3).astype(np.int32)
    want = oracle.pool_scores(s32.astype(np.float64), wl.cu_seqlens_k, kernel, mode)
    dev = DeviceWorkload(wl)
    dev.poison()
    pooled = torch.full(s32.shape, float("nan"), dtype=torch.float32, device="cuda")
    pdd.select_topk_pooled(torch.from_numpy(s32).cuda(), dev.cu_k, dev.max_k, dev.k_keep, dev.cu_keep, dev.total_keep,
                           dev.idx, dev.mask, kernel, pdd.POOL_MAX if mode == "max" else pdd.POOL_AVG, pooled,
                           dev.cand_b, dev.cand_e, wl.cu_seqlens_k)
    got = pooled.cpu().numpy().astype(np.float64)
    # one fp32 chain of up to 1025 additions of values of size 1, times 1 / kernel (itself rounded)
    atol = 0 if mode == "max" else kernel * 2.0 ** -24 * np.abs(s32).max() * 2
    np.testing.assert_allclose(got, want, rtol=0, atol=atol)
    check_selection(got, dev.idx.cpu().numpy(), dev.mask.cpu().numpy(), wl, -1, "pooled")


@pytest.mark.parametrize("mode", ["max", "avg"])
@pytest.mark.parametrize("n", [2, 300, 4097, 20000, 33000])
def test_pooled_selection_ranks_what_it_returns(n, mode):
    """The ranking and the pooled scores that the call returns agree where scores are infinite or NaN, in rows
    that stay in registers and in longer ones: a maximum over NaN alone is NaN (its key lies above
    +infinity's), at the ends of the row too.  Exact, from the returned scores' bits."""
    rng, kernel = np.random.default_rng(n), 7
    s32 = rng.normal(size=(2, n)).astype(np.float32)
    s32[:, rng.integers(0, n, n // 50)] = -np.inf
    s32[1, rng.integers(0, n, n // 90)] = np.inf
    for at in [0, n - 9] + list(rng.integers(0, n, n // 200)):
        s32[:, max(at, 0):at + int(rng.integers(5, 20))] = np.nan
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    cu = np.array([0, n], dtype=np.int32)
    for k in sorted({1, n // 20 + 1, n // 2, n}):
        idx = torch.full((2, k), -7, dtype=torch.int32, device="cuda")
        mask = torch.full((2, n), 9, dtype=torch.uint8, device="cuda")
        pooled = torch.zeros((2, n), dtype=torch.float32, device="cuda")
        pdd.select_topk_pooled(dev(s32), dev(cu), n, dev(np.array([k], dtype=np.int32)), dev(np.array([0, k], dtype=np.int32)), k,
                               idx, mask, kernel, pdd.POOL_MAX if mode == "max" else pdd.POOL_AVG, pooled, None, None, cu)
        got = pooled.cpu().numpy()
        pad = np.pad(np.isnan(s32), ((0, 0), (3, 3)), constant_values=mode == "max")
        all_or_any = np.lib.stride_tricks.sliding_window_view(pad, kernel, axis=1)
        if mode == "max":
            assert np.array_equal(np.isnan(got), all_or_any.all(-1))
        else:                                                    # infinities of both signs make a NaN as well
            assert np.isnan(got[all_or_any.any(-1)]).all()
        bits = (got + np.float32(0)).view(np.int32).astype(np.int64)
        key = np.where(bits < 0, -1 - bits, bits + 2 ** 31)
        want = np.sort(np.argsort(-key, axis=1, kind="stable")[:, :k], axis=1)
        assert np.array_equal(idx.cpu().numpy(), want), k
        assert all(np.array_equal(np.flatnonzero(mask[g].cpu().numpy()), want[g]) for g in range(2)), k


# ------------------------------------------------- sentence-level selection
def _sentence_split(rng, lo, hi, mean_len, with_empty):
    """Ends of sentences tiling [lo, hi): geometric lengths, optionally a few empty ones."""
    ends, x = [], lo
    while x < hi:
        x = min(hi, x + int(rng.geometric(1.0 / mean_len)))
        ends.append(x)
        if with_empty and rng.random() < 0.05:
            ends.append(x)
    return ends


def _oracle_keep_on_kernel_scores(got_sc, cu, cu_sent, ends, budget, cb):
    """The oracle's sentence ranking applied to the fp32 sentence scores the kernel ranked: a
    token-score array that holds each sentence's score on its first token and zero elsewhere
    sums (mode "sum") to exactly that score, so oracle.select_sentences ranks the kernel's own
    values with the real sentence lengths and budget."""
    H = got_sc.shape[0]
    tok = np.zeros((H, int(cu[-1])), dtype=np.float64)
    for b in range(len(cu) - 1):
        start = int(cb[b])
        for s_ in range(cu_sent[b], cu_sent[b + 1]):
            if ends[s_] > start:
                tok[:, cu[b] + start] = got_sc[:, s_]
            else:
                assert (got_sc[:, s_] == 0).all()           # an empty sentence scores zero
            start = int(ends[s_])
    sc, keep, mask, kept = oracle.select_sentences(tok, cu, cu_sent, ends, budget, "sum", cb)
    assert np.array_equal(sc, got_sc)
    return keep, mask, kept


@pytest.mark.parametrize("mode", ["sum", "mean"])
@pytest.mark.parametrize("exact_scores", [True, False])
def test_select_sentences(mode, exact_scores):
    rng = np.random.default_rng(31)
    lens = [900, 1, 0, 37, 32768, 9000]
    heads = 2
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cb = np.array([16, 0, 0, 5, 128, 0], dtype=np.int32)
    ce = [880, 1, 0, 30, 32768 - 64, 9000]
    mean_len = [18, 1, 1, 4, 24, 1.2]                   # the last sequence has ~7500 sentences
    ends, cu_sent = [], [0]
    for b in range(len(lens)):
        e = _sentence_split(rng, int(cb[b]), ce[b], mean_len[b], b != 5) if ce[b] > cb[b] else []
        ends += e
        cu_sent.append(len(ends))
    ends = np.array(ends, dtype=np.int32)
    cu_sent = np.array(cu_sent, dtype=np.int32)
    max_sent = int(np.diff(cu_sent).max())
    assert 4096 < max_sent <= 8192
    budget = np.array([300, 1, 0, 10, 3276, 4000], dtype=np.int32)
    if exact_scores:      # multiples of 1/64 with short sums: fp32 sums and means of sums are order-free
        s32 = (rng.integers(0, 64, size=(heads, int(cu[-1]))) / 64.0).astype(np.float32)
        if mode == "mean":                              # a mean is one rounded division on both sides
            pass
    else:
        s32 = (rng.random((heads, int(cu[-1]))) ** 6).astype(np.float32)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    n_sent = len(ends)
    sscore = torch.full((heads, n_sent), float("nan"), dtype=torch.float32, device="cuda")
    skeep = torch.full((heads, n_sent), 7, dtype=torch.uint8, device="cuda")
    mask = torch.full((heads, int(cu[-1])), 7, dtype=torch.uint8, device="cuda")
    kept = torch.full((heads, len(lens)), -1, dtype=torch.int32, device="cuda")
    pdd.select_sentences(d(s32), d(cu), max(lens), d(cu_sent), d(ends), max_sent, d(budget),
                         pdd.SENT_SUM if mode == "sum" else pdd.SENT_MEAN, d(cb), sscore, skeep, mask, kept, cu)
    torch.cuda.synchronize()
    got_sc = sscore.cpu().numpy().astype(np.float64)
    want_sc, want_keep, want_mask, want_kept = oracle.select_sentences(
        s32.astype(np.float64), cu, cu_sent, ends, budget, mode, cb)
    np.testing.assert_allclose(got_sc, want_sc, rtol=2e-6, atol=1e-12)
    if exact_scores and mode == "sum":
        assert np.array_equal(got_sc, want_sc)
        assert np.array_equal(skeep.cpu().numpy(), want_keep)
    # the decision is exact on the sentence scores the kernel ranked (fp32, as the kernel holds them)
    kf = skeep.cpu().numpy()
    x_keep, x_mask, x_kept = _oracle_keep_on_kernel_scores(got_sc, cu, cu_sent, ends, budget, cb)
    assert np.array_equal(kf, x_keep)
    assert np.array_equal(mask.cpu().numpy(), x_mask)             # token mask = expansion of the flags
    assert np.array_equal(kept.cpu().numpy(), x_kept) and (x_kept <= budget[None, :]).all()
    # against the fp64 oracle: identical up to sentences whose scores tie within fp32 rounding
    diff = kf != want_keep
    if diff.any():
        assert not exact_scores or mode == "mean"
        for g, s in zip(*np.nonzero(diff)):
            b = int(np.searchsorted(cu_sent, s, side="right") - 1)
            sl = slice(cu_sent[b], cu_sent[b + 1])
            others = np.delete(want_sc[g, sl], s - cu_sent[b])
            assert np.min(np.abs(others - want_sc[g, s])) <= 4e-6 * max(abs(want_sc[g, s]), 1e-30), (g, s)


@pytest.mark.parametrize("mean_len,levels", [(24.0, 8), (1.0, 1), (9.0, 64), (400.0, 3)])
def test_select_sentences_with_ties(mean_len, levels):
    """Sentences that tie in score (few score levels, down to one for the whole row, where the index
    alone decides), 1 to 8192 of them, budgets from nothing to everything, rows of more than 32768
    tokens and rows that start at any byte of the mask: exact, because every score is a small integer."""
    rng = np.random.default_rng(int(mean_len) + levels)
    lens = [70001, 1025, 3, 64, 33000, 8191, 500]
    counts = [min(8192, max(1, int(n / mean_len))) for n in lens]
    cb = [0, 1, 0, 0, 7, 0, 499]
    ends, cu_sent = [], [0]
    for n, c, lo in zip(lens, counts, cb):
        ends.append(np.sort(rng.integers(lo, n + 1, size=c)))      # empty sentences among them
        cu_sent.append(cu_sent[-1] + c)
    ends = np.concatenate(ends).astype(np.int32)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cu_sent = np.array(cu_sent, dtype=np.int32)
    cb = np.array(cb, dtype=np.int32)
    # one score per sentence on its first token: the sum is that score
    heads = 2
    tok = np.zeros((heads, int(cu[-1])), dtype=np.float32)
    for b in range(len(lens)):
        start = int(cb[b])
        for s in range(cu_sent[b], cu_sent[b + 1]):
            if ends[s] > start:
                tok[:, cu[b] + start] = rng.integers(0, levels, size=heads) - levels // 2
            start = int(ends[s])
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    for share in (0.0, 0.001, 0.3, 0.9, 1.0):
        budget = np.array([int(share * n) for n in lens], dtype=np.int32)
        skeep = torch.full((heads, len(ends)), 7, dtype=torch.uint8, device="cuda")
        mask = torch.full((heads, int(cu[-1])), 7, dtype=torch.uint8, device="cuda")
        kept = torch.full((heads, len(lens)), -1, dtype=torch.int32, device="cuda")
        pdd.select_sentences(d(tok), d(cu), max(lens), d(cu_sent), d(ends), max(counts), d(budget), pdd.SENT_SUM,
                             d(cb), None, skeep, mask, kept, cu)
        torch.cuda.synchronize()
        _, w_keep, w_mask, w_kept = oracle.select_sentences(tok.astype(np.float64), cu, cu_sent, ends, budget, "sum", cb)
        assert np.array_equal(skeep.cpu().numpy(), w_keep), share
        assert np.array_equal(mask.cpu().numpy(), w_mask), share
        assert np.array_equal(kept.cpu().numpy(), w_kept), share


# --------------------------------------------------- cross-layer aggregation
@pytest.mark.parametrize("layers,heads,total_k", [(33, 3, 130), (1, 9, 4099), (40, 1, 16385), (7, 17, 63), (5, 2, 70001),
                                                  (1, 1, 5), (2, 3, 1027), (3, 1, 70001), (3, 16, 65539), (5, 64, 65541)])
@pytest.mark.parametrize("reduce_heads", [False, True])
def test_aggregate_scores_shapes(layers, heads, total_k, reduce_heads):
    """Layers shared by 1 to 16 waves, workgroups of one to four runs of tokens, 1 to 4 tokens per lane, one to
    eight loads in flight, rows that start at any 4-byte address.
    Positive terms: an fp32 sum of n of them, weighted, is within (n + 2) 2^-24 of its value."""
    rng = np.random.default_rng(layers)
    s32 = rng.random((layers, heads, total_k)).astype(np.float32)
    w32 = (rng.random(layers) + 0.5).astype(np.float32)
    out = torch.full((1 if reduce_heads else heads, total_k), 2.0, dtype=torch.float32, device="cuda")
    for accumulate in (False, True):
        pdd.aggregate_scores(torch.from_numpy(s32).cuda(), out, torch.from_numpy(w32).cuda(), reduce_heads, accumulate)
        torch.cuda.synchronize()
        want = oracle.aggregate_scores(s32, w32, reduce_heads) * (2 if accumulate else 1)
        n = 2 * layers * (heads if reduce_heads else 1) + 2
        np.testing.assert_allclose(out.cpu().numpy().astype(np.float64), want, rtol=n * 2.0 ** -24)


@pytest.mark.parametrize("total_k,reduce_heads", [(32768, False), (32768, True), (1003, False), (1003, True)])
def test_aggregate_scores(total_k, reduce_heads):
    rng = np.random.default_rng(17)
    n_layers, heads = 6, 8
    s32 = (rng.random((n_layers, heads, total_k)) ** 6).astype(np.float32)
    w32 = rng.random(n_layers).astype(np.float32)
    rows = 1 if reduce_heads else heads
    want = oracle.aggregate_scores(s32, w32, reduce_heads)
    out = torch.full((rows, total_k), float("nan"), dtype=torch.float32, device="cuda")
    sd = torch.from_numpy(s32).cuda()
    pdd.aggregate_scores(sd, out, torch.from_numpy(w32).cuda(), reduce_heads)
    torch.cuda.synchronize()
    np.testing.assert_allclose(out.cpu().numpy().astype(np.float64), want, rtol=2e-6, atol=1e-12)
    # unweighted, one layer at a time into the same buffer == all layers at once
    out2 = torch.zeros((rows, total_k), dtype=torch.float32, device="cuda")
    for l in range(n_layers):
        pdd.aggregate_scores(sd[l:l + 1], out2, None, reduce_heads, accumulate=True)
    torch.cuda.synchronize()
    np.testing.assert_allclose(out2.cpu().numpy().astype(np.float64),
                               oracle.aggregate_scores(s32, None, reduce_heads), rtol=2e-6, atol=1e-12)
    # a strided layer view (every second layer of the stack)
    out3 = torch.empty((rows, total_k), dtype=torch.float32, device="cuda")
    pdd.aggregate_scores(sd[::2], out3, None, reduce_heads)
    torch.cuda.synchronize()
    np.testing.assert_allclose(out3.cpu().numpy().astype(np.float64),
                               oracle.aggregate_scores(s32[::2], None, reduce_heads), rtol=2e-6, atol=1e-12)


# ------------------------------------ the refinement stages chained end to end
def test_refinement_pipeline_end_to_end():
    """Attention + importance -> sum over heads -> sentence-level selection under the token
    budget floor(r * l) with a protected prefix and suffix -> bit stream.  Importance parity is
    covered above; here every later stage is checked against the oracle applied to the scores
    the previous GPU stage produced."""
    wl = W.make_custom("t", [1500, 333], None, 8, 2, 128, 48, "1/4", seed=9)
    dev = DeviceWorkload(wl)
    dev.step()
    imp = dev.imp                                               # [Hkv, total_k] fp32 on the GPU
    oI = oracle.importance(wl.q, wl.k, wl.cu_seqlens_q, wl.cu_seqlens_k, wl.scale, wl.window)
    rel_close(imp.cpu().numpy().astype(np.float64), oI, "importance")
    # all heads into one score row
    allh = torch.empty((1, wl.total_k), dtype=torch.float32, device="cuda")
    pdd.aggregate_scores(imp.view(1, wl.n_kv_heads, wl.total_k), allh, None, reduce_heads=True)
    torch.cuda.synchronize()
    want_all = oracle.aggregate_scores(imp.cpu().numpy()[None], None, True)
    np.testing.assert_allclose(allh.cpu().numpy().astype(np.float64), want_all, rtol=2e-6, atol=1e-12)
    # sentences over the content part, prefix of 20 and suffix of 12 tokens protected
    rng = np.random.default_rng(4)
    lens = np.diff(wl.cu_seqlens_k)
    cb = np.array([20, 20], dtype=np.int32)
    ends, cu_sent = [], [0]
    for b in range(2):
        ends += _sentence_split(rng, 20, int(lens[b]) - 12, 15, False)
        cu_sent.append(len(ends))
    ends = np.array(ends, dtype=np.int32)
    cu_sent = np.array(cu_sent, dtype=np.int32)
    budget = np.array([int(lens[b]) // 4 for b in range(2)], dtype=np.int32)   # floor(r * l), r = 1/4
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    sscore = torch.empty((1, len(ends)), dtype=torch.float32, device="cuda")
    skeep = torch.empty((1, len(ends)), dtype=torch.uint8, device="cuda")
    mask = torch.full((1, wl.total_k), 9, dtype=torch.uint8, device="cuda")
    kept = torch.empty((1, 2), dtype=torch.int32, device="cuda")
    pdd.select_sentences(allh, dev.cu_k, dev.max_k, d(cu_sent), d(ends), int(np.diff(cu_sent).max()),
                         d(budget), pdd.SENT_MEAN, d(cb), sscore, skeep, mask, kept, wl.cu_seqlens_k)
    torch.cuda.synchronize()
    w_sc, w_keep, w_mask, w_kept = oracle.select_sentences(
        allh.cpu().numpy().astype(np.float64), wl.cu_seqlens_k, cu_sent, ends, budget, "mean", cb)
    np.testing.assert_allclose(sscore.cpu().numpy().astype(np.float64), w_sc, rtol=2e-6, atol=1e-12)
    # the decision, on the sentence scores the kernel ranked
    g_sc = sscore.cpu().numpy().astype(np.float64)
    x_keep, x_mask, x_kept = _oracle_keep_on_kernel_scores(g_sc, wl.cu_seqlens_k, cu_sent, ends, budget, cb)
    assert np.array_equal(skeep.cpu().numpy(), x_keep)
    assert np.array_equal(mask.cpu().numpy(), x_mask)
    assert np.array_equal(kept.cpu().numpy(), x_kept) and (x_kept <= budget[None, :]).all()
    for b in range(2):
        seq = mask.cpu().numpy()[0, wl.cu_seqlens_k[b]:wl.cu_seqlens_k[b + 1]]
        assert seq[:20].sum() == 0 and seq[int(lens[b]) - 12:].sum() == 0 and seq.sum() == int(x_kept[0, b])
    # bit stream of the token mask
    want_bits, cu_bytes = oracle.pack_mask(mask.cpu().numpy(), wl.cu_seqlens_k)
    bits = torch.empty((1, int(cu_bytes[-1])), dtype=torch.uint8, device="cuda")
    pdd.pack_mask(mask, dev.cu_k, dev.max_k, d(cu_bytes), int(cu_bytes[-1]), bits)
    torch.cuda.synchronize()
    assert np.array_equal(bits.cpu().numpy(), want_bits)
