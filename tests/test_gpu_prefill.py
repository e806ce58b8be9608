"""GPU parity of the prefill path (MFMA tiles): local sink+window attention, the dense comparison,
and the retrieval heads' chunk kernel, against the CPU oracle row by row."""
import re

import numpy as np
import pytest
import torch

from oracle import rtp_oracle as orc
from paper_2605_16928_amd import rtp, workloads as wl
from gpu_util import (DEV, PrefillRun, prefill_oracle_inputs, check_out, check_out_any, reported_sets, count_range, i32, i64,
                      layer_desc_of, ws_alloc)

pytestmark = pytest.mark.gpu


def _cases():
    return {
        # two query tiles with a ragged tail, band crossing several key tiles, sinks outside the band
        "small": dict(),
        # first chunk of a sequence: queries below the sink count, below one key tile
        "first_chunk": dict(chunk_start=0, T=130, seed=42),
        # window narrower than a key tile, no sinks
        "narrow": dict(chunk_start=300, T=100, sink=0, window=30, seed=43),
        # more sinks than one key tile holds
        "many_sinks": dict(chunk_start=900, T=64, sink=70, window=100, seed=44),
        # window wider than the context: local == dense
        "wide": dict(chunk_start=200, T=129, sink=4, window=4096, seed=45),
        # group sizes 1 and 8
        "g1": dict(n_q_heads=4, n_kv_heads=4, ret_heads=(2,), chunk_start=257, T=65, seed=46),
        "g8": dict(n_q_heads=16, n_kv_heads=2, ret_heads=(0, 8), chunk_start=1000, T=96, seed=47),
        # a single query
        "one_query": dict(chunk_start=333, T=1, seed=48),
        # fp16 attention tensors
        "small_f16": dict(seed=49, kv_dtype="fp16"),
        "g8_f16": dict(n_q_heads=16, n_kv_heads=2, ret_heads=(0, 8), chunk_start=1000, T=96, seed=50, kv_dtype="fp16"),
        "first_chunk_f16": dict(chunk_start=0, T=130, seed=51, kv_dtype="fp16"),
    }


@pytest.mark.parametrize("name", list(_cases()))
def test_prefill_local_dense_and_retrieval_p1(name):
    print(f"[case] prefill {name}", flush=True)
    w = wl.small_prefill(DEV, **_cases()[name])
    L = w.layer
    run = PrefillRun(w)
    oi = prefill_oracle_inputs(w)
    rows = [(t, h) for t in range(w.T) for h in range(L.n_q_heads)]

    # local heads + retrieval heads with p = 1 (the paper's prefill rule) fill the whole output
    run.out.fill_(9.0)
    run.local_attn()
    run.sparse_prefill(p=1.0)
    torch.cuda.synchronize()
    out = run.out.float().cpu().numpy().astype(np.float64)
    lse = run.lse.cpu().numpy()
    ref = orc.prefill_rows(rows=rows, p=1.0, **oi)
    o_ref = np.zeros_like(out)
    l_ref = np.zeros_like(lse)
    for r in ref:
        o_ref[r["t"], r["h"]] = r["out"]
        l_ref[r["t"], r["h"]] = r["lse"]
    check_out(out, o_ref, f"{name} local + retrieval(p=1)", tight="mfma")
    assert np.allclose(lse, l_ref, atol=3e-3, rtol=0)

    # dense comparison over all heads
    dout = torch.zeros_like(run.out)
    dlse = torch.zeros_like(run.lse)
    run.dense_attn(dout, dlse)
    torch.cuda.synchronize()
    dref = orc.dense_rows(rows=rows, q_bits=oi["q_bits"], K_bits=oi["K_bits"], V_bits=oi["V_bits"],
                          chunk_start=w.chunk_start, n_q_heads=L.n_q_heads, n_kv_heads=L.n_kv_heads, kv_dtype=L.kv_dtype)
    o_ref = np.zeros_like(out)
    for r in dref:
        o_ref[r["t"], r["h"]] = r["out"]
    check_out(dout.float().cpu().numpy().astype(np.float64), o_ref, f"{name} dense", tight="mfma")


def test_prefill_two_sequences_and_interleaved_kv():
    """B = 2 packed sequences with different chunk positions; K|V interleaved rows."""
    print("[case] prefill two sequences / interleaved", flush=True)
    d = wl.small_decode(DEV, seed=51, ctx=(900, 1300), sink=4, window=200, n_planted=0)
    L = d.layer
    n_q = 70
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    q = torch.randn((2, n_q, L.n_q_heads, 128), generator=g, device=DEV).to(torch.bfloat16)
    q_start = [900 - n_q, 1300 - n_q - 37]
    desc = layer_desc_of(L)
    out = torch.zeros((2, n_q, L.n_q_heads, 128), dtype=torch.bfloat16, device=DEV)
    dout = torch.zeros_like(out)
    ws = ws_alloc(rtp.rtp_local_attn_workspace_bytes(desc, 2, n_q, 1300))
    kv = torch.cat([d.K, d.V], dim=2).contiguous()
    T = d.T_tot
    rtp.rtp_local_attn(desc, q, kv.data_ptr(), kv.data_ptr() + 256, 256, T * 256, i64(d.seq_start), i32(d.ctx_len),
                       i32(q_start), 2, n_q, 1300, out, None, ws)
    rtp.rtp_dense_attn(desc, q, d.K, d.V, 128, T * 128, i64(d.seq_start), i32(d.ctx_len), i32(q_start), 2, n_q, 1300,
                       dout, None, ws)
    torch.cuda.synchronize()
    Kb, Vb, qb = wl.bf16_bits(d.K), wl.bf16_bits(d.V), wl.bf16_bits(q)
    local_heads = [h for h in range(L.n_q_heads) if h not in L.ret_heads]
    for b in range(2):
        s0, n = d.seq_start[b], d.ctx_len[b]
        common = dict(q_bits=qb[b], K_bits=Kb[:, s0:s0 + n], V_bits=Vb[:, s0:s0 + n], chunk_start=q_start[b],
                      n_q_heads=L.n_q_heads, n_kv_heads=L.n_kv_heads)
        rows = [(t, h) for t in range(n_q) for h in local_heads]
        ref = orc.prefill_rows(rows=rows, kI_bits=None, ret_heads=L.ret_heads, sink=L.sink, window=L.window, p=1.0,
                               **common)
        got = out[b].float().cpu().numpy().astype(np.float64)
        for r in ref:
            check_out(got[r["t"], r["h"]], r["out"], f"local b{b} t{r['t']} h{r['h']}", tight="mfma")
        for h in L.ret_heads:
            assert np.all(got[:, h] == 0)                       # retrieval rows untouched by the local call
        rows = [(t, h) for t in range(n_q) for h in range(L.n_q_heads)]
        dref = orc.dense_rows(rows=rows, **common)
        dgot = dout[b].float().cpu().numpy().astype(np.float64)
        for r in dref:
            check_out(dgot[r["t"], r["h"]], r["out"], f"dense b{b} t{r['t']} h{r['h']}", tight="mfma")


def _dense_vs_oracle(w, what):
    L = w.layer
    run = PrefillRun(w)
    oi = prefill_oracle_inputs(w)
    rows = [(t, h) for t in range(w.T) for h in range(L.n_q_heads)]
    dout = torch.zeros_like(run.out)
    dlse = torch.zeros_like(run.lse)
    run.dense_attn(dout, dlse)
    torch.cuda.synchronize()
    dref = orc.dense_rows(rows=rows, q_bits=oi["q_bits"], K_bits=oi["K_bits"], V_bits=oi["V_bits"],
                          chunk_start=w.chunk_start, n_q_heads=L.n_q_heads, n_kv_heads=L.n_kv_heads)
    got = dout.float().cpu().numpy().astype(np.float64)
    o_ref = np.zeros_like(got)
    for r in dref:
        o_ref[r["t"], r["h"]] = r["out"]
    assert np.isfinite(got).all(), what
    check_out(got, o_ref, what, tight="mfma")


def test_dense_prefill_scores_far_above_the_first_tile():
    """The dense kernel takes every query's reference maximum from the first key tile.  Here the late
    keys score ~90 (natural units) above it: exp overflows against that reference and the workgroup
    has to notice and repeat its keys with the running-maximum recurrence."""
    print("[case] dense prefill, reference outrun upwards", flush=True)
    w = wl.small_prefill(DEV, seed=91, chunk_start=600, T=150)
    w.q[:] = 2.0
    w.K[:, 300:, :] = 4.0                     # q.k * scale = 128 * 8 / sqrt(128) ~ 90.5 for keys >= 300
    _dense_vs_oracle(w, "reference outrun upwards")


def test_dense_prefill_reference_above_every_visible_score():
    """First chunk: keys 32..63 score ~90 above the rest but the first 32 queries cannot see them, so
    their reference (taken over the whole first tile, masks ignored) is far above everything they
    attend to; their probabilities underflow and the repeat pass has to produce them."""
    print("[case] dense prefill, reference outrun downwards", flush=True)
    w = wl.small_prefill(DEV, seed=92, chunk_start=0, T=100)
    w.q[:] = 2.0
    w.K[:, :, :] = (torch.randn_like(w.K.float()) * 0.05).to(w.K.dtype)
    w.K[:, 32:64, :] = 4.0
    _dense_vs_oracle(w, "reference outrun downwards")


# ---------------------------------------------------------------------------------------------
# per-query top-p in prefill (p < 1)
# ---------------------------------------------------------------------------------------------
FINE = 2.0 ** -17           # threshold resolution of the prefill selector (score units)
BAND = 3e-5                 # fp32 rounding of (max - score) and of the MFMA index scores


def _sparse_cases():
    return {
        "small_p90": (dict(), 0.9),
        "small_p50": (dict(seed=61), 0.5),
        "small_p999": (dict(seed=62), 0.999),
        "first_chunk": (dict(chunk_start=0, T=150, seed=63), 0.9),
        "proj": (dict(index_mode="proj", chunk_start=500, T=70, seed=64), 0.8),
        "zipf_g8": (dict(n_q_heads=16, n_kv_heads=2, ret_heads=(0, 8), chunk_start=1800, T=96, seed=65, zipf=1.1), 0.9),
        "p_to_one": (dict(chunk_start=300, T=40, seed=66), 0.9999999),
        # fp16 attention tensors: the matrix-core variants on binary16 operands
        "small_f16": (dict(seed=68, kv_dtype="fp16"), 0.9),
        "g8_f16": (dict(n_q_heads=16, n_kv_heads=2, ret_heads=(0, 8), chunk_start=1800, T=96, seed=69, kv_dtype="fp16"), 0.8),
    }


@pytest.mark.parametrize("name", list(_sparse_cases()))
def test_sparse_prefill_matches_oracle(name):
    print(f"[case] sparse prefill {name}", flush=True)
    kw, p = _sparse_cases()[name]
    w = wl.small_prefill(DEV, p=p, **kw)
    _check_sparse_prefill(w, name, p)


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp16"])
def test_sparse_prefill_peaked_law_skips_key_tiles(kv_dtype):
    """A peaked indexer law: the own cluster of 8 tokens holds nearly all the mass, runs of 32 queries share a
    cluster, so p = 0.9 keeps a handful of tokens per query and most 64-key tiles hold no kept pair of a whole
    query tile.  The attention launch leaves those tiles out; everything it reports still matches the oracle,
    and the tile statistics show the skipping."""
    print(f"[case] sparse prefill, peaked law, {kv_dtype}", flush=True)
    w = wl.small_prefill(DEV, p=0.9, chunk_start=9000, T=600, seed=70, own_frac=0.99, pick_run=32, kv_dtype=kv_dtype)
    cnt = _check_sparse_prefill(w, f"peaked_{kv_dtype}", 0.9)
    assert np.median(cnt) <= 16
    run = PrefillRun(w)
    run.sparse_prefill(p=0.9)
    visited, causal = run.tile_stats()
    n_ret = w.layer.n_ret
    assert causal == n_ret * sum((9000 + min(t0 + 256, 600) - 1) // 64 + 1 for t0 in range(0, 600, 256))
    print(f"   tiles visited {visited} of {causal}", flush=True)
    assert 0 < visited < causal // 2
    # p close to 1 reaches every tile: the list is the whole causal range again
    run.sparse_prefill(p=0.9999999)
    assert run.tile_stats()[0] > causal // 2


def test_sparse_prefill_key_ranges_without_a_kept_key():
    """Long context, few heads: the launch cuts every query tile's key range in two, and with a small p the
    few kept tokens of a query leave whole ranges empty -- a legitimate zero partial, not a failed reference."""
    print("[case] sparse prefill, empty key ranges", flush=True)
    w = wl.small_prefill(DEV, p=0.3, chunk_start=6000, T=64, seed=67)
    cnt = _check_sparse_prefill(w, "empty_ranges", 0.3)
    assert cnt.min() < 64                     # some query keeps less than one tile's worth of keys


def test_sparse_prefill_reference_outrun_repeats_exactly():
    """The selecting mode on inputs whose late keys score ~90 above the first tile: the fixed reference
    overflows and the workgroup repeats its keys with the running maximum, keep test included."""
    print("[case] sparse prefill, reference outrun upwards", flush=True)
    w = wl.small_prefill(DEV, p=0.9, chunk_start=600, T=150, seed=93)
    w.q[:] = 2.0
    w.K[:, 300:, :] = 4.0
    _check_sparse_prefill(w, "sparse_outrun", 0.9)


def _check_sparse_prefill(w, name, p):
    L = w.layer
    run = PrefillRun(w)
    oi = prefill_oracle_inputs(w)
    run.out.fill_(5.0)
    run.sparse_prefill()
    torch.cuda.synchronize()
    out = run.out.float().cpu().numpy().astype(np.float64)
    tau, cnt, mass = run.tau.cpu().numpy(), run.count.cpu().numpy(), run.mass.cpu().numpy()
    p32 = float(np.float32(p))
    rows = [(t, h) for t in range(w.T) for h in L.ret_heads]
    ref = orc.prefill_rows(rows=rows, p=p32, **oi)
    sc = 1.0 / np.sqrt(128.0)
    worst = 0.0
    for r in ref:
        t, h, m = r["t"], r["h"], r["m"]
        j = L.ret_heads.index(h)
        s = r["scores"]
        wgt = np.exp(s - s.max())
        Z = wgt.sum()
        tg = float(tau[j, t])
        # (a) the kept set reaches p, and the threshold is never above the exact one
        keep = s > tg
        amb = np.abs(s - tg) <= BAND
        assert tg <= r["sel"]["tau"] + BAND, f"{name} t{t} h{h}: threshold {tg} above the exact {r['sel']['tau']}"
        assert wgt[keep | amb].sum() / Z >= p32 - 1e-6, f"{name} t{t} h{h}: kept mass below p"
        # (b) ... and not lower than one fine bin
        if np.isfinite(tg):
            above = s > tg + FINE + BAND
            assert wgt[above].sum() / Z < p32 + 1e-6, \
                f"{name} t{t} h{h}: threshold {tg} is more than one fine bin below the exact one"
        # (c) statistics
        assert abs(int(cnt[j, t]) - int(keep.sum())) <= int(amb.sum()), f"{name} t{t} h{h}: count {cnt[j, t]} vs {keep.sum()}"
        assert abs(mass[j, t] - wgt[keep].sum() / Z) <= 1e-5 + wgt[amb].sum() / Z
        # (d) attention over the set the library kept.  The reported threshold and the kernel's keep test are
        # fp32 roundings of the same bound, so a token whose fp64 score lies within the band of the reported
        # threshold may be on either side: any set between {s > tau + band} and {s >= tau - band} is a legal
        # reading of the report.  The reported count says how many band tokens are in; the test is
        # monotone in the score, so they are the highest-scoring ones (band tokens whose scores differ by less
        # than fp32 resolves may swap: then any choice of that many is accepted).
        kvh = h // (L.n_q_heads // L.n_kv_heads)

        def att(ids):
            return orc.attend(oi["q_bits"][t, h], oi["K_bits"][kvh, :m + 1], oi["V_bits"][kvh, :m + 1], ids, sc, L.kv_dtype)[0]

        def att_abs(ids):
            return orc.attend(oi["q_bits"][t, h], oi["K_bits"][kvh, :m + 1], oi["V_bits"][kvh, :m + 1] & 0x7fff, ids, sc,
                              L.kv_dtype)[0]

        worst = max(worst, check_out_any(out[t, h], reported_sets(s, tg, int(cnt[j, t]), BAND, f"{name} t{t} h{h}"), att,
                                         f"{name} t{t} h{h} (same set)", att_abs))
        # (e) end to end against the exact top-p set: the stated tolerance.  Tokens within 1e-5 of the
        # exact threshold may legitimately differ; rows that have such a token are only held to (d).
        near = np.abs(s - r["sel"]["tau"]) <= 1e-5 * max(1.0, abs(r["sel"]["tau"]))
        if near.sum() <= 1:
            k_lo, k_hi = count_range(s, p32)
            assert k_lo <= int(cnt[j, t]) <= k_hi, f"{name} t{t} h{h}: set differs ({cnt[j, t]} kept, exact {r['sel']['count']})"
            if k_lo == k_hi:
                assert int(cnt[j, t]) == r["sel"]["count"]
                check_out(out[t, h], r["out"], f"{name} t{t} h{h} (exact top-p)", tight=False)
    for h in range(L.n_q_heads):
        if h not in L.ret_heads:
            assert np.all(out[:, h] == 5.0)
    print(f"   worst abs err vs same-set oracle {worst:.2e}; kept tokens min/mean/max "
          f"{cnt.min()}/{cnt.mean():.1f}/{cnt.max()}", flush=True)
    return cnt


def test_sparse_prefill_p1_statistics_and_dense_equivalence():
    """p = 1 with statistics requested runs the selecting kernel with nothing to select:
    the dense path's output up to rounding (the two kernels block the keys differently),
    count = m + 1, mass = 1."""
    print("[case] sparse prefill p=1 statistics", flush=True)
    w = wl.small_prefill(DEV, seed=71, chunk_start=260, T=90)
    run = PrefillRun(w)
    L = w.layer
    run.sparse_prefill(p=1.0)
    torch.cuda.synchronize()
    a = run.out.clone()
    cnt = run.count.cpu().numpy()
    assert np.array_equal(cnt, np.tile(w.chunk_start + np.arange(w.T) + 1, (L.n_ret, 1)))
    assert np.all(run.mass.cpu().numpy() == 1.0)
    dout = torch.zeros_like(run.out)
    run.dense_attn(dout)
    torch.cuda.synchronize()
    ga = a[:, L.ret_heads].float().cpu().numpy().astype(np.float64)
    gd = dout[:, L.ret_heads].float().cpu().numpy().astype(np.float64)
    assert (np.abs(ga - gd) <= 2e-3 + 2.0 ** -7 * np.abs(gd)).all(), np.abs(ga - gd).max()


def test_retrieval_dense_split_keys_matches_unsplit():
    """Few heads and a long context: the dense rule cuts every query tile's key range into parts and
    merges them.  With a workspace the split path runs, without one the unsplit path: same result."""
    print("[case] dense retrieval rule with key-range splits", flush=True)
    w = wl.small_prefill(DEV, seed=81, chunk_start=6000, T=130, n_q_heads=4, n_kv_heads=2, ret_heads=(1,))
    run = PrefillRun(w)
    L = w.layer
    need = rtp.rtp_sparse_attn_prefill_workspace_bytes(run.desc, w.T, w.chunk_start)
    assert need > L.n_ret * w.T * 132 * 4            # room for at least two partials per row
    a = torch.zeros_like(run.out)
    b = torch.zeros_like(run.out)
    la, lb = torch.zeros_like(run.lse), torch.zeros_like(run.lse)
    args = (run.desc, w.qI, w.q, None, w.kI, w.N * 16, run.Kp, run.Vp, run.rs, run.hs, w.chunk_start, w.T, 1.0)
    rtp.rtp_sparse_attn_prefill(*args, a, la, None, None, None, run.ws)
    rtp.rtp_sparse_attn_prefill(*args, b, lb, None, None, None, None)
    torch.cuda.synchronize()
    oi = prefill_oracle_inputs(w)
    rows = [(t, 1) for t in range(w.T)]
    ref = orc.dense_rows(rows=rows, q_bits=oi["q_bits"], K_bits=oi["K_bits"], V_bits=oi["V_bits"],
                         chunk_start=w.chunk_start, n_q_heads=L.n_q_heads, n_kv_heads=L.n_kv_heads)
    ga = a.float().cpu().numpy().astype(np.float64)
    gb = b.float().cpu().numpy().astype(np.float64)
    for r in ref:
        check_out(ga[r["t"], 1], r["out"], "split", tight="mfma")
        check_out(gb[r["t"], 1], r["out"], "unsplit", tight="mfma")
        assert abs(la[r["t"], 1].item() - r["lse"]) < 3e-3 and abs(lb[r["t"], 1].item() - r["lse"]) < 3e-3


@pytest.mark.parametrize("scale,p", [(2.0, 0.999999), (2.5, 0.9999999), (3.0, 0.999999)])
def test_sparse_prefill_threshold_far_below_the_row_maximum(scale, p):
    """Score rows whose bulk lies 13 to 22 below the row maximum, with p so close to 1 that the threshold falls
    into that bulk: the search's first digit covers 15.875 below its reference, so it must lower the reference
    and repeat for such queries instead of keeping every candidate (fp32 p cannot push a threshold much deeper
    than that at these lengths; every repeat runs the same code).  Checked like every
    other case: exact sets away from the threshold band, counts, masses, attention over the kept set."""
    print(f"[case] sparse prefill, threshold far below the maximum, scale {scale} p {p}", flush=True)
    w = wl.small_prefill("cpu", p=p, chunk_start=2500, T=96, seed=97)
    w.layer.index_scale = scale
    w = w.to(DEV)
    cnt = _check_sparse_prefill(w, f"far_{scale}", p)
    # the case does what it is meant to: for most queries the threshold lies more than 15.875 below the maximum,
    # and the kept set is neither tiny nor the whole candidate set
    run = PrefillRun(w)
    run.sparse_prefill()
    torch.cuda.synchronize()
    oi = prefill_oracle_inputs(w)
    ref = orc.prefill_rows(rows=[(t, w.layer.ret_heads[0]) for t in range(0, w.T, 8)], p=float(np.float32(p)), **oi)
    deep = [r["sel"]["smax"] - r["sel"]["tau"] for r in ref]
    assert max(deep) > 15.875 and (scale > 2.75 or np.median(deep) > 15.875), deep
    assert all(r["sel"]["count"] < r["m"] + 1 for r in ref)


@pytest.mark.parametrize("chunk_start,T", [(0, 1), (0, 33), (255, 31), (256, 65), (1000, 97), (2047, 33)])
def test_sparse_prefill_partial_query_groups(chunk_start, T):
    """Chunks whose last 32-query group is partial, with causal ranges that end on, one before and one behind the edges of
    the search's key tiles (32) and rounds (256): the group's spare lanes repeat its last query and must leave no trace."""
    print(f"[case] sparse prefill, partial group, T {T} behind {chunk_start}", flush=True)
    w = wl.small_prefill(DEV, p=0.9, chunk_start=chunk_start, T=T, seed=101 + T)
    _check_sparse_prefill(w, f"partial_{chunk_start}_{T}", 0.9)


@pytest.mark.parametrize("chunk_start,T", [(0, 257), (63, 130), (191, 257), (256, 256), (449, 65), (640, 511)])
@pytest.mark.parametrize("kv_dtype", ["bf16", "fp16"])
def test_prefill_dense_rule_around_the_steady_loop(chunk_start, T, kv_dtype):
    """Key ranges whose mask-free part begins, ends or is cut short on, before and behind the edges of the 64-key tiles
    and of the 256-query tiles; partial query tiles leave waves without a query.  The dense rule with statistics."""
    print(f"[case] dense rule, T {T} behind {chunk_start}, {kv_dtype}", flush=True)
    w = wl.small_prefill(DEV, chunk_start=chunk_start, T=T, n_q_heads=4, n_kv_heads=2, ret_heads=(1,), seed=111 + T, kv_dtype=kv_dtype)
    _check_dense_rule(w, f"{chunk_start}+{T}")


@pytest.mark.parametrize("chunk_start,T", [(9000, 1), (4000, 64), (3000, 300), (505, 9)])
def test_prefill_dense_rule_short_chunks_in_many_key_ranges(chunk_start, T):
    """Short chunks cut their keys into up to 64 ranges (512 keys at the least) and merge them."""
    print(f"[case] dense rule, T {T} behind {chunk_start}", flush=True)
    w = wl.small_prefill(DEV, chunk_start=chunk_start, T=T, n_q_heads=4, n_kv_heads=2, ret_heads=(1,), seed=131 + T)
    _check_dense_rule(w, f"{chunk_start}+{T}")
    _check_sparse_prefill(w, f"{chunk_start}+{T}", 0.9)


def _check_dense_rule(w, what):
    L = w.layer
    run = PrefillRun(w)
    run.sparse_prefill(p=1.0)
    torch.cuda.synchronize()
    oi = prefill_oracle_inputs(w)
    rows = [(t, h) for t in range(w.T) for h in L.ret_heads]
    ref = orc.dense_rows(rows=rows, q_bits=oi["q_bits"], K_bits=oi["K_bits"], V_bits=oi["V_bits"], chunk_start=w.chunk_start,
                         n_q_heads=L.n_q_heads, n_kv_heads=L.n_kv_heads, kv_dtype=L.kv_dtype)
    got = run.out.float().cpu().numpy().astype(np.float64)
    lse = run.lse.cpu().numpy()
    for r in ref:
        check_out(got[r["t"], r["h"]], r["out"], f"{what} t{r['t']} h{r['h']}", tight="mfma")
        assert abs(lse[r["t"], r["h"]] - r["lse"]) < 3e-3
    assert np.array_equal(run.count.cpu().numpy(), np.tile(w.chunk_start + np.arange(w.T) + 1, (L.n_ret, 1)))
    assert np.all(run.mass.cpu().numpy() == 1.0) and np.all(np.isneginf(run.tau.cpu().numpy()))


@pytest.mark.parametrize("chunk_start,T,kw,p", [
    (13000, 1, {}, 0.9), (20000, 33, {}, 0.8), (14335, 40, dict(own_frac=0.99, pick_run=32), 0.9), (30001, 70, dict(index_mode="proj"), 0.95)])
def test_sparse_prefill_sliced_search(chunk_start, T, kw, p):
    """Short chunks behind long prefixes: the threshold search runs as one launch per sweep with several workgroups per
    query group, whose maxima and histograms the next launch merges."""
    print(f"[case] sliced search, T {T} behind {chunk_start}", flush=True)
    w = wl.small_prefill(DEV, p=p, chunk_start=chunk_start, T=T, seed=151 + T, n_q_heads=4, n_kv_heads=2, ret_heads=(1,), **kw)
    _check_sparse_prefill(w, f"sliced_{chunk_start}_{T}", p)


@pytest.mark.parametrize("chunk_start,T,kw,p", [
    (5087, 33, {}, 0.9), (5120, 1, {}, 0.8), (5121, 65, dict(own_frac=0.99, pick_run=32), 0.9), (8200, 97, dict(index_mode="proj"), 0.95),
    (6000, 40, dict(index_scale=2.5), 0.999999),
    (11487, 33, {}, 0.9), (11520, 1, {}, 0.8), (11521, 65, dict(own_frac=0.99, pick_run=32), 0.9), (12000, 97, dict(index_mode="proj"), 0.95),
    (11600, 40, dict(index_scale=2.5), 0.999999)])
def test_sparse_prefill_search_in_large_workgroups(chunk_start, T, kw, p):
    """Few query groups with keys for more than 90 rounds of tiles: workgroups of sixteen waves, on either side of the first such
    length, and with thresholds in the open-ended bin."""
    print(f"[case] search in large workgroups, T {T} behind {chunk_start}", flush=True)
    kw = dict(kw)
    scale = kw.pop("index_scale", None)
    w = wl.small_prefill("cpu", p=p, chunk_start=chunk_start, T=T, seed=161 + T, n_q_heads=4, n_kv_heads=2, ret_heads=(1,), **kw)
    if scale:
        w.layer.index_scale = scale
    w = w.to(DEV)
    names = _launches(PrefillRun(w).sparse_prefill)
    assert any("kSelThreadsFew" in n for n in names) == (chunk_start + T > 90 * 128) and not any("<0>" in n for n in names), names
    _check_sparse_prefill(w, f"large_{chunk_start}_{T}", p)


def test_sparse_prefill_sliced_search_with_a_threshold_in_the_open_ended_bin():
    """A query group with a threshold more than 15.875 below a row maximum leaves the sliced form: its last launch searches
    the group from the start."""
    print("[case] sliced search, threshold far below the maximum", flush=True)
    w = wl.small_prefill("cpu", p=0.999999, chunk_start=13000, T=40, seed=98)
    w.layer.index_scale = 2.5
    _check_sparse_prefill(w.to(DEV), "sliced_far", 0.999999)


@pytest.mark.parametrize("p", [0.9, 1.0])
@pytest.mark.parametrize("kv_dtype", ["bf16", "fp16"])
def test_prefill_log_sums_of_masked_rows_carry_no_rounding(p, kv_dtype):
    """Rows whose keys all lie in a part's first block or in masked ones sum unrounded probabilities: at most 32 terms in fp32
    against a score error of 128 products in fp32 (|score| < 16), so 2^-24 * (32 + 128 * 16) < 1.3e-4 at the very worst; the
    rounded sum of a few bf16 terms is off by up to 2^-9 = 2e-3 (fp16: 2^-12 = 2.4e-4)."""
    print(f"[case] log-sums of masked rows, p {p}, {kv_dtype}", flush=True)
    w = wl.small_prefill(DEV, chunk_start=0, T=172, seed=161, n_q_heads=4, n_kv_heads=2, ret_heads=(1, 2), kv_dtype=kv_dtype)
    run = PrefillRun(w)
    run.sparse_prefill(p=p)
    torch.cuda.synchronize()
    lse = run.lse.cpu().numpy().astype(np.float64)
    ref = orc.prefill_rows(rows=[(t, h) for t in range(32) for h in w.layer.ret_heads], p=p, **prefill_oracle_inputs(w))
    worst = max(abs(lse[r["t"], r["h"]] - r["lse"]) for r in ref)
    assert worst < 1.3e-4, worst


@pytest.mark.parametrize("chunk_start,window", [(200, 64), (255, 40), (128, 100), (191, 30)])
def test_local_prefill_infinite_value_of_the_last_key(chunk_start, window):
    """The rows a ragged last tile stages past the last key take part with probability 0 and value 0: an infinite value of the
    last key gives its own query infinity, not NaN."""
    print(f"[case] local prefill, infinite last value, {chunk_start}", flush=True)
    w = wl.small_prefill(DEV, chunk_start=chunk_start, T=1, sink=4, window=window, seed=171)
    w.V[:, chunk_start, 3] = float("inf")
    run = PrefillRun(w)
    run.local_attn()
    torch.cuda.synchronize()
    heads = [h for h in range(w.layer.n_q_heads) if h not in w.layer.ret_heads]
    out = run.out[0, heads].float()
    assert torch.isposinf(out[:, 3]).all()
    assert torch.isfinite(out[:, :3]).all() and torch.isfinite(out[:, 4:]).all()


def _launches(call):
    rtp.rtp_profile_start(64)
    try:
        call()
    finally:
        recorded = rtp.rtp_profile_stop(64)
    return [name for name, _ in recorded]


@pytest.mark.parametrize("p", [0.9, 1.0])
def test_short_chunk_in_the_workspace_of_a_whole_chunk(p):
    """The last 333 queries of a prompt in the workspace that served its chunks of 4096: the same launches as with a workspace of
    their own, and the same result.  In the least workspace there is the short chunk runs in fewer workgroups: the same selection,
    outputs that differ by the order of fp32 sums and one rounding to 16 bits."""
    print(f"[case] short chunk, long chunk's workspace, p {p}", flush=True)
    w = wl.make_prefill("tail", wl.Layer(32, 8, [0, 8, 16, 24], sink=4, window=256), 131072, 333, p, 181, DEV, cluster_len=32)
    run = PrefillRun(w)
    size = lambda T, c: rtp.rtp_sparse_attn_prefill_workspace_bytes(run.desc, T, c)
    args = (run.desc, w.qI, w.q, None, w.kI, w.N * 16, run.Kp, run.Vp, run.rs, run.hs, w.chunk_start, w.T, p)

    def go(n_bytes):
        ws = torch.full((n_bytes,), 0xAB, dtype=torch.uint8, device=DEV)
        o, l = torch.zeros_like(run.out), torch.zeros_like(run.lse)
        st = (run.tau, run.count, run.mass) if p < 1.0 else (None, None, None)
        for t in st:
            if t is not None:
                t.fill_(-5)
        names = _launches(lambda: rtp.rtp_sparse_attn_prefill(*args, o, l, *st, ws))
        torch.cuda.synchronize()
        return names, o[:, w.layer.ret_heads].float(), l[:, w.layer.ret_heads], [t.clone() for t in st if t is not None]

    one_range = w.layer.n_ret * w.T * 132 * 4
    if p < 1.0:
        lo, hi = 0, size(w.T, w.chunk_start) // 256          # the least accepted size, in units of 256 bytes
        while hi - lo > 1:
            mid = (lo + hi) // 2
            try:
                go(mid * 256)
                hi = mid
            except rtp.RtpError as e:
                assert e.code == rtp.RTP_ERR_WORKSPACE
                lo = mid
        least = hi * 256
        assert least < 7 << 20
    else:
        least = 8 * one_range
    own, whole, small = go(size(w.T, w.chunk_start)), go(size(4096, w.chunk_start - 4096)), go(least)
    assert own[0] == whole[0] and any("combine" in n for n in own[0])
    assert sum("select_kernel" in n for n in own[0]) == (5 if p < 1.0 else 0)
    for names, o, l, st in (whole, small):
        assert any("combine" in n for n in names)
        assert ((o - own[1]).abs() <= 2.0 ** -7 * torch.maximum(o.abs(), own[1].abs()) + 1e-5).all()
        assert (l - own[2]).abs().max() < 1e-4
        if p < 1.0:
            assert torch.equal(st[0], own[3][0]) and torch.equal(st[1], own[3][1]) and (st[2] - own[3][2]).abs().max() < 1e-6
    if p >= 1.0:
        names, o, l, _ = go(one_range - 256)
        assert len(names) == 1 and (l - own[2]).abs().max() < 1e-4


@pytest.mark.parametrize("T,heads", [(1, 64), (130, 64), (600, 64), (560, 128)])
@pytest.mark.parametrize("kv_dtype", ["bf16", "fp16"])
def test_local_prefill_one_and_two_wave_groups(T, heads, kv_dtype):
    """Launches of at most one workgroup per compute unit give a query's band to two groups of waves, larger ones (600 and 560
    queries of 60 and 120 heads: more than 256 workgroups) to one: odd and even numbers of key tiles, ragged ends, sinks outside
    the band."""
    print(f"[case] local prefill, T {T}, {heads} heads, {kv_dtype}", flush=True)
    w = wl.small_prefill(DEV, chunk_start=777, T=T, n_q_heads=heads, n_kv_heads=heads // 8, ret_heads=tuple(range(0, heads, heads // 4)),
                         sink=4, window=300, seed=191 + T, kv_dtype=kv_dtype)
    L = w.layer
    run = PrefillRun(w)
    run.out.fill_(5.0)
    run.local_attn()
    torch.cuda.synchronize()
    local = [h for h in range(heads) if h not in L.ret_heads]
    rows = [(t, h) for t in sorted({0, 1, 31, 32, 127, 128, 129, T // 2, T - 2, T - 1} & set(range(T))) for h in local[::17] + local[-1:]]
    ref = orc.prefill_rows(rows=rows, p=1.0, **prefill_oracle_inputs(w))
    got, lse = run.out.float().cpu().numpy().astype(np.float64), run.lse.cpu().numpy()
    for r in ref:
        check_out(got[r["t"], r["h"]], r["out"], f"t{r['t']} h{r['h']}", tight="mfma")
        assert abs(lse[r["t"], r["h"]] - r["lse"]) < 3e-3
    assert (run.out[:, list(L.ret_heads)] == 5.0).all()


@pytest.mark.parametrize("chunk_start,T,sink,window,groups", [
    (0, 192, 4, 512, 1), (0, 193, 4, 512, 2),                              # three and four tiles of keys in all
    (5000, 1, 4, 65, 1), (5000, 1, 4, 66, 2), (5000, 1, 0, 129, 1),        # by the window: one sink tile and two or three of the band
    (5000, 128, 4, 2, 2), (100, 64, 64, 16, 1), (6, 3, 0, 0x7fffffff, 1)])
def test_local_prefill_groups_by_the_tiles_of_a_band(chunk_start, T, sink, window, groups):
    """Bands that cannot have four key tiles are left to one group of waves."""
    print(f"[case] band of {T} queries behind {chunk_start}, {sink} + {window}", flush=True)
    w = wl.small_prefill(DEV, chunk_start=chunk_start, T=T, n_q_heads=8, n_kv_heads=2, ret_heads=(1,), sink=sink, window=window, seed=311)
    run = PrefillRun(w)
    names = _launches(run.local_attn)
    assert len(names) == 1 and names[0].strip("()").endswith(f", {groups}>"), names
    torch.cuda.synchronize()
    rows = [(t, h) for t in sorted({0, T // 2, T - 1}) for h in (0, 7)]
    got = run.out.float().cpu().numpy().astype(np.float64)
    for r in orc.prefill_rows(rows=rows, p=1.0, **prefill_oracle_inputs(w)):
        check_out(got[r["t"], r["h"]], r["out"], f"t{r['t']} h{r['h']}", tight="mfma")


def _check_rounded_probabilities(o, o1, kv_dtype="bf16"):
    """Two results [.., 128] of the same set, probabilities rounded to 8 bits (fp16: 11) against different references.  A rounding is off by at most
    2^-8 of the value, evenly spread at the worst: the difference of two has a standard deviation of at most 2^-8 sqrt(2/3) of the probability, and a
    sum over keys with independent values that share of the row's root mean square.  Six of these, and the results' own roundings."""
    ulp = 2.0 ** (-11 if kv_dtype == "fp16" else -8)
    rms = torch.maximum(o.pow(2).mean(-1, keepdim=True), o1.pow(2).mean(-1, keepdim=True)).sqrt()
    worst = ((o - o1).abs() - 2 * ulp * torch.maximum(o.abs(), o1.abs())).div(rms).max().item()
    print(f"   differ by {worst / ulp:.2f} roundings of a row's rms", flush=True)
    assert worst <= 6 * (2.0 / 3.0) ** 0.5 * ulp


@pytest.mark.parametrize("chunk_start,T,heads,kw,kv_dtype", [
    (1 << 20, 513, (1, 2, 3), {}, "bf16"),                                   # one query past two tiles of 256; a sliced search
    (520001, 777, (0, 2, 3), dict(own_frac=0.99, pick_run=32), "fp16"),     # three heads; a ragged last tile and group
    (150000, 2113, (0, 1, 2, 3), dict(zipf=1.1, cluster_len=32), "bf16"),   # whole rows, more groups than compute units
    (62000, 4600, (0, 1, 2, 3), {}, "bf16"),                             # two blocks, the second one short
    (700000, 600, (1, 2, 3), dict(index_mode="proj"), "bf16"),                   # every query keeps much: nothing to regroup
    (150000, 2100, (0, 1, 2, 3), dict(own_frac=0.97, pick_run=64, tokens_per_cluster=32768, q_noise=0.1), "bf16"),   # every one little
    (800000, 530, (1, 2, 3), dict(index_scale=2.5, p=0.999999), "bf16"),         # thresholds in the open-ended bin, sliced
    (150000, 2081, (0, 1, 2, 3), dict(index_scale=2.5, p=0.999999), "bf16"),    # and in whole rows
    (150000, 2113, (0, 1, 2, 3), dict(recent=9.0), "fp16")])               # some queries find the token before them far above the rest
def test_sparse_prefill_with_regrouped_queries(chunk_start, T, heads, kw, kv_dtype):
    """Chunks behind a long prefix take their queries by how much they keep.  In the least workspace there is, they take them by
    position: the same selection, and outputs that differ by the order of fp32 sums and the rounding of probabilities to 16 bits
    against other references."""
    print(f"[case] regrouped queries, T {T} behind {chunk_start}, {heads}, {kw}, {kv_dtype}", flush=True)
    kw = dict(kw)
    scale, p, recent = kw.pop("index_scale", None), kw.pop("p", 0.9), kw.pop("recent", 0.0)
    w = wl.make_prefill("regrouped", wl.Layer(8, 4, list(heads), sink=4, window=256, kv_dtype=kv_dtype), chunk_start, T, p, 211 + T, DEV, **kw)
    if scale:
        w.layer.index_scale = scale
    for t in range(5, T, 64) if recent else ():
        for j, h in ((0, 0), (2, 2)):                              # (two query heads to a KV head)
            q, n = w.q[t, h].float(), chunk_start + t - 1
            w.K[h // 2, n] = ((4.0 + recent) * 128 ** 0.5 * q / q.dot(q)).to(w.K.dtype)
            w.kI[j, n] = (w.kI[j].float().norm(dim=-1).max() * w.qI[j, t].float() / w.qI[j, t].float().norm()).to(torch.bfloat16)
    run = PrefillRun(w)
    need = rtp.rtp_sparse_attn_prefill_workspace_bytes(run.desc, T, chunk_start)

    def go(n_bytes):
        ws = torch.full((n_bytes,), 0xAB, dtype=torch.uint8, device=DEV)
        o, l = torch.zeros_like(run.out), torch.zeros_like(run.lse)
        st = [torch.full_like(t, -5) for t in (run.tau, run.count, run.mass)]
        q_in = w.q_pre if w.WQ is not None else w.qI
        names = _launches(lambda: rtp.rtp_sparse_attn_prefill(run.desc, q_in, w.q, w.WQ, w.kI, w.N * 16, run.Kp, run.Vp, run.rs, run.hs,
                                                              chunk_start, T, p, o, l, *st, ws))
        torch.cuda.synchronize()
        return names, o[:, w.layer.ret_heads].float(), l[:, w.layer.ret_heads], st

    lo, hi = 0, need // 256
    while hi - lo > 1:
        mid = (lo + hi) // 2
        try:
            go(mid * 256)
            hi = mid
        except rtp.RtpError as e:
            assert e.code == rtp.RTP_ERR_WORKSPACE
            lo = mid
    names, o, l, st = go(need)
    plain, o1, l1, st1 = go(hi * 256)
    assert any("order_kernel" in n for n in names) and not any("order_kernel" in n for n in plain), (names, plain)
    assert torch.equal(st[0], st1[0]) and torch.equal(st[1], st1[1]) and (st[2] - st1[2]).abs().max() < 1e-6
    _check_rounded_probabilities(o, o1, kv_dtype)
    assert (l - l1).abs().max() < 6e-3
    assert st[1].min() >= 1


@pytest.mark.parametrize("scale", [1.0, 2.0, 3.0, 4.0, 6.0, 10.0, 24.0])
def test_sparse_prefill_fp16_few_kept_keys_far_from_the_first_tile(scale):
    """fp16 probabilities against a range's reference, its first tile's best: queries that keep a handful of keys, with scores all around it
    (scale 1: within +-4; 2 to 4: probabilities down to subnormals; 24: far above and below, where the exact pass has to take over)."""
    print(f"[case] fp16, few kept keys, scale {scale}", flush=True)
    w = wl.small_prefill("cpu", chunk_start=3000, T=70, seed=231, n_q_heads=4, n_kv_heads=2, ret_heads=(1,), own_frac=0.99, pick_run=32, kv_dtype="fp16")
    w.q.mul_(scale)
    _check_sparse_prefill(w.to(DEV), f"f16_few_{scale}", 0.9)


@pytest.mark.parametrize("chunk_start,T,sink,window,bound,kv_dtype", [
    (5000, 1, 4, 1000, 0, "bf16"), (5000, 130, 4, 1000, 0, "fp16"), (3001, 333, 70, 2048, 0, "bf16"), (2047, 97, 0, 1025, 0, "bf16"),
    (0, 40, 4, 2048, 4096, "bf16"),            # one tile of keys where the bound allows for thirty: empty ranges
    (63, 257, 4, 4096, 8192, "fp16"), (1100, 64, 1200, 100, 0, "bf16")])
def test_local_prefill_key_ranges(chunk_start, T, sink, window, bound, kv_dtype):
    """Few workgroups and long bands: the key tiles are cut into ranges whose partial results a second launch merges.  Without room
    for them in the workspace, one range; both against the oracle, and retrieval heads untouched."""
    print(f"[case] local prefill in ranges, T {T} behind {chunk_start}, {sink} + {window}, {kv_dtype}", flush=True)
    w = wl.small_prefill(DEV, chunk_start=chunk_start, T=T, n_q_heads=8, n_kv_heads=2, ret_heads=(1,), sink=sink, window=window, seed=411 + T,
                         kv_dtype=kv_dtype)
    L, run = w.layer, PrefillRun(w)
    max_ctx = max(w.N, bound)
    need = rtp.rtp_local_attn_workspace_bytes(run.desc, 1, T, max_ctx)
    rows = [(t, h) for t in sorted({0, 1, 31, 32, 127, 128, T // 2, T - 1} & set(range(T))) for h in (0, 2, 7)]
    ref = orc.prefill_rows(rows=rows, p=1.0, **prefill_oracle_inputs(w))
    for n_bytes in (need, 256):
        ws = torch.full((max(n_bytes, 256),), 0xAB, dtype=torch.uint8, device=DEV)
        out, lse = torch.full_like(run.out, 5.0), torch.full_like(run.lse, 5.0)
        names = _launches(lambda: rtp.rtp_local_attn(run.desc, w.q, run.Kp, run.Vp, run.rs, run.hs, run.seq_start, run.ctx_len, run.q_start,
                                                     1, T, max_ctx, out, lse, ws))
        torch.cuda.synchronize()
        assert any("combine" in n for n in names) == (n_bytes == need), names
        got, l = out.float().cpu().numpy().astype(np.float64), lse.cpu().numpy()
        for r in ref:
            check_out(got[r["t"], r["h"]], r["out"], f"t{r['t']} h{r['h']}", tight="mfma")
            assert abs(l[r["t"], r["h"]] - r["lse"]) < 3e-3
        assert (out[:, 1] == 5.0).all() and (lse[:, 1] == 5.0).all()


def test_local_band_between_a_search_and_its_tile_stats():
    """The local band's partials go to a workspace of their own: the figures of the search before it stay."""
    w = wl.small_prefill(DEV, chunk_start=3001, T=333, n_q_heads=8, n_kv_heads=2, ret_heads=(1,), sink=4, window=2048, seed=417)
    run = PrefillRun(w)
    run.sparse_prefill(p=0.5)
    stats = run.tile_stats()
    assert any("combine" in n for n in _launches(run.local_attn))
    assert 0 < stats[0] <= stats[1] and run.tile_stats() == stats


@pytest.mark.parametrize("chunk_start,T,window", [(200, 1153, 200), (199, 1153, 200), (3000, 1281, 90), (0, 1281, 2048)])
def test_local_prefill_of_more_workgroups_than_compute_units(chunk_start, T, window):
    """A KV head to a die from the first chunk on whose window lies before it; KV heads of four local heads and of three, a last tile of
    one query, a number of workgroups that eight does not divide."""
    print(f"[case] local prefill of many workgroups, T {T} behind {chunk_start}, window {window}", flush=True)
    w = wl.small_prefill(DEV, chunk_start=chunk_start, T=T, n_q_heads=32, n_kv_heads=8, ret_heads=(1, 9, 31), sink=4, window=window, seed=431 + T)
    run = PrefillRun(w)
    out, lse = torch.full_like(run.out, 5.0), torch.full_like(run.lse, 5.0)
    run.local_attn(out, lse)
    torch.cuda.synchronize()
    got, l = out.float().cpu().numpy().astype(np.float64), lse.cpu().numpy()
    rows = [(t, h) for t in (0, 127, 128, T // 2, T - 1) for h in (0, 3, 8, 16, 30)]
    for r in orc.prefill_rows(rows=rows, p=1.0, **prefill_oracle_inputs(w)):
        check_out(got[r["t"], r["h"]], r["out"], f"t{r['t']} h{r['h']}", tight="mfma")
        assert abs(l[r["t"], r["h"]] - r["lse"]) < 3e-3
    local = [h for h in range(32) if h not in (1, 9, 31)]
    assert (lse[:, local] != 5.0).all() and (out[:, [1, 9, 31]] == 5.0).all()


def _in_least_workspace(run, p):
    """The chunk in the smallest workspace that is accepted: the kernels launched and out, lse, tau, count, mass."""
    w = run.w
    o, l = torch.zeros_like(run.out), torch.zeros_like(run.lse)
    st = [torch.full_like(t, -5) for t in (run.tau, run.count, run.mass)]

    def go(n_bytes):
        ws = torch.full((n_bytes,), 0xAB, dtype=torch.uint8, device=DEV)
        return _launches(lambda: rtp.rtp_sparse_attn_prefill(run.desc, w.q_pre if w.WQ is not None else w.qI, w.q, w.WQ, w.kI, w.N * 16, run.Kp,
                                                             run.Vp, run.rs, run.hs, w.chunk_start, w.T, p, o, l, *st, ws))

    with pytest.raises(rtp.RtpError) as e:
        go(256)
    assert e.value.code == rtp.RTP_ERR_WORKSPACE
    names = go(int(re.search(r"workspace of (\d+) bytes", str(e.value)).group(1)))
    torch.cuda.synchronize()
    return names, (o, l, *st)


@pytest.mark.parametrize("T,planned", [(8192, True), (8193, False)])
def test_sparse_prefill_up_to_the_lists_that_are_planned_and_past_them(T, planned):
    """64 retrieval heads with as many queries as the attention launch's work is planned for, and one more: that call is the one of the least
    workspace there is, bit for bit.  Rows of either end and of the middle are the oracle's."""
    print(f"[case] sparse prefill, 64 retrieval heads, T {T}", flush=True)
    w = wl.make_prefill("many_lists", wl.Layer(64, 8, list(range(64)), sink=4, window=256), 60000, T, 0.9, 307, DEV, zipf=1.1)
    run = PrefillRun(w)
    assert any("order_kernel" in n for n in _launches(run.sparse_prefill)) == planned
    torch.cuda.synchronize()
    full = [t.clone() for t in (run.out, run.lse, run.tau, run.count, run.mass)]
    names, least = _in_least_workspace(run, w.p)
    assert not any("order_kernel" in n for n in names), names
    for what, a, b in list(zip(("out", "lse", "tau", "count", "mass"), full, least))[2 if planned else 0:]:
        assert torch.equal(a, b) or what == "mass" and (a - b).abs().max() < 1e-6, what
    _check_rounded_probabilities(full[0].float(), least[0].float())
    assert (full[1] - least[1]).abs().max() < 6e-3
    out, lse, cnt = full[0].float().cpu().numpy().astype(np.float64), full[1].cpu().numpy(), full[3].cpu().numpy()
    rows = [(t, h) for t in (0, 255, 4100, T - 1) for h in (0, 37, 63)]
    for r in orc.prefill_rows(rows=rows, p=float(np.float32(w.p)), **prefill_oracle_inputs(w)):
        t, h = r["t"], r["h"]
        k_lo, k_hi = count_range(r["scores"], float(np.float32(w.p)))
        # (a token within 2^-17 below the threshold is kept as well)
        near = int((np.abs(r["scores"] - r["sel"]["tau"]) <= BAND).sum())
        assert k_lo - near <= cnt[h, t] <= k_hi + near, (t, h, cnt[h, t], r["sel"]["count"])
        check_out(out[t, h], r["out"], f"t{t} h{h}", tight=False)
        assert abs(lse[t, h] - r["lse"]) < 6e-3


@pytest.mark.parametrize("p", [0.9, 1.0])
@pytest.mark.parametrize("above", [2.0, 4.0, 6.0, 9.0, 12.0, 20.0])
def test_fp16_prefill_one_recent_key_far_above_the_rest(above, p):
    """fp16 probabilities end at 65504.  One query finds one key of its own diagonal block `above` units over anything else it sees; every
    other query is ordinary, so that no other row makes the workgroup repeat its keys."""
    print(f"[case] fp16, one recent key {above} above, p {p}", flush=True)
    w = wl.small_prefill("cpu", chunk_start=3000, T=70, seed=233, n_q_heads=4, n_kv_heads=2, ret_heads=(1,), kv_dtype="fp16", p=p)
    t, n, h = 40, 3035, 1
    q = w.q[t, h].float()
    best = (w.K[0].float() @ q).max() / 128 ** 0.5
    w.K[0, n] = ((best + above) * 128 ** 0.5 * q / q.dot(q)).to(w.K.dtype)
    w.kI[0, n] = (4.0 * w.qI[0, t].float() / w.qI[0, t].float().norm()).to(torch.bfloat16)   # (kept by the query, whoever else keeps it)
    w = w.to(DEV)
    if p < 1.0:
        _check_sparse_prefill(w, f"f16_recent_{above}", p)
        return
    run = PrefillRun(w)
    run.sparse_prefill()
    torch.cuda.synchronize()
    got = run.out.float().cpu().numpy().astype(np.float64)
    for r in orc.prefill_rows(rows=[(i, h) for i in range(w.T)], p=1.0, **prefill_oracle_inputs(w)):
        check_out(got[r["t"], h], r["out"], f"t{r['t']}", tight="mfma")


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("chunk_start", [500, 3000])          # one range of keys; several, of which the first holds the key
def test_sparse_prefill_a_kept_key_that_is_not_a_number(chunk_start, kv_dtype):
    """A kept key whose scores are not a number, alone in its block of 32: its row says so (no finite log-sum, no output), whoever else is kept."""
    print(f"[case] sparse prefill, NaN in a kept key, {chunk_start}, {kv_dtype}", flush=True)
    w = wl.small_prefill("cpu", chunk_start=chunk_start, T=1, seed=235, n_q_heads=4, n_kv_heads=2, ret_heads=(1,), kv_dtype=kv_dtype, p=0.9)
    kept = orc.prefill_rows(rows=[(0, 1)], p=0.9, **prefill_oracle_inputs(w))[0]["sel"]["idx"]
    alone = [n for n in kept if (np.asarray(kept) // 32 == n // 32).sum() == 1]
    assert len(kept) > 1 and alone
    w.K[0, min(alone)] = float("nan")
    run = PrefillRun(w.to(DEV))
    run.sparse_prefill()
    torch.cuda.synchronize()
    assert int(run.count[0, 0]) == len(kept)
    assert not torch.isfinite(run.lse[0, 1]) and not (run.out[0, 1] != 0).any()
