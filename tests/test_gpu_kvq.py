"""Parity of the 2-bit token-wise K/V path (records, attention on records, decode step on records) against the
CPU oracle, through the C ABI.

Bars: alpha bit-equal; records against the oracle's fields (the quantisation function in fp64 with true
divisions) under the rule of helpers.records_agree: sign bytes equal, stored parameters and 2-bit codes equal
except where the exact value lies within the library's binary32 rounding error of an fp16 rounding boundary /
of a half-integer of t = (x - zp) / qs (the exceptions are counted and printed; where nothing is near a tie the
records are byte-for-byte the oracle's); attention within the same bars as the 16-bit path (1e-5 relative for
fp32 output) against the oracle's fp64 attention over the dequantised rows of THE SAME records; top-k sets as in
the 16-bit decode step (scoring does not depend on the K/V format).
"""
import numpy as np
import pytest
import torch

import sik_workloads as W
from helpers import dev, records_agree, topk_sets_agree
from test_gpu_parity import TDT, check_attention, cfg_small, sync

pytestmark = pytest.mark.gpu

import paper_2603_14224_amd as sik  # noqa: E402


class Q2State:
    """One layer's cache quantised by the oracle (fields + packed records) and mirrored on the device."""

    def __init__(self, cfg, oracle, capacity=None, seq_len=None, offset_std=0.0, out_dtype=None, K=None, V=None):
        self.cfg, self.o = cfg, oracle
        if K is None:
            K, V = W.make_cache(cfg, capacity=capacity, channel_offset_std=offset_std)
        self.K, self.V = K, V
        B, H, cap, D = K.shape
        self.sl = np.full(B, cfg.context, np.int32) if seq_len is None else np.asarray(seq_len, np.int32)
        self.mu, self.codes, self.cb, _ = oracle.fit(K, cfg.dtype, self.sl)
        self.alpha, self.qkv = oracle.fit_q2(K, V, cfg.dtype, self.sl, self.mu)
        self.layout = sik.make_layout(B, H, cfg.n_q_heads, D, cap, TDT[cfg.dtype], out_dtype)
        self.dK, self.dV = dev(K, cfg.dtype), dev(V, cfg.dtype)
        self.dsl = torch.from_numpy(self.sl.copy()).cuda()
        self.dmu = torch.from_numpy(self.mu).cuda()
        self.dcb = torch.from_numpy(self.cb).cuda()
        self.dcodes = torch.from_numpy(self.codes).cuda()
        self.ws = sik.alloc_workspace(self.layout, min(cfg.top_k, cap))

    def records(self):
        return self.o.pack_records(self.codes, self.qkv)


def check_records(st, got, K, V, qkv, codes, ranges, label):
    """got against the oracle's fields on token ranges [(b, t0, t1)]; prints the near-tie exceptions."""
    exc = np.zeros(4, np.int64)
    for b, t0, t1 in ranges:
        exc += records_agree(st.o, got, K, V, st.cfg.dtype, st.mu, st.alpha, codes, qkv, b, t0, t1)
    print(f"{label}: {exc[0]} of {exc[2]} parameters and {exc[1]} of {exc[3]} codes inside the near-tie band")
    return exc


def adopt_appended_records(oracle, kvq, kn, vn, dtype, mu, alpha, codes, qkv, sl):
    """After a decode step that appended token sl[b] - 1 on both sides: the library's record of that token must
    match the oracle's (already in qkv) under the near-tie rule; the oracle then takes over the library's own row,
    so that attention is compared on identical records."""
    B, Hkv = kn.shape[0], kn.shape[1]
    for b in range(B):
        t = int(sl[b]) - 1
        row = np.zeros((B, Hkv, 1, 128), np.uint8)
        row[b] = kvq[b, :, t:t + 1].cpu().numpy()
        records_agree(oracle, row, kn[:, :, None, :], vn[:, :, None, :], dtype, mu, alpha, codes, qkv, b, t, t + 1,
                      base=t)
        _, one = oracle.unpack_records(row[b:b + 1])
        for f in ("kq", "vq", "kpar", "vpar"):
            getattr(qkv, f)[b, :, t] = getattr(one, f)[0, :, 0]


def gpu_fit(st):
    dal = torch.full(st.mu.shape, -1.0, device="cuda")
    kvq = sik.alloc_kvq(st.layout)
    sik.sik_quantize_kv(st.layout, st.dK, st.dV, st.dsl, 0, 0, sik.SIK_Q_FIT, st.dmu, dal, kvq)
    sync()
    return dal, kvq


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("offset", [0.0, 1.5])
def test_fit_alpha_and_records_match_oracle(oracle, dtype, offset):
    cfg = cfg_small(batch=2, n_kv_heads=3, n_q_heads=6, context=1337, top_k=64, dtype=dtype, seed=41)
    st = Q2State(cfg, oracle, capacity=1400, seq_len=[1337, 801], offset_std=offset)
    dal, kvq = gpu_fit(st)
    assert np.array_equal(dal.cpu().numpy(), st.alpha)
    got = kvq.cpu().numpy()
    exc = check_records(st, got, st.K, st.V, st.qkv, st.codes, [(b, 0, int(L)) for b, L in enumerate(st.sl)],
                        f"fit {dtype} offset {offset}")
    assert exc[0] <= exc[2] // 500 and exc[1] <= exc[3] // 10000     # a sliver, not a systematic difference
    for b, L in enumerate(st.sl):
        assert not got[b, :, L:].any()            # records beyond seq_len are not written
    assert sik.sik_kvq_bytes(st.layout) == got.nbytes


def test_encode_range_against_frozen_parameters(oracle):
    # tokens appended later may exceed the fitted range (|K - mu| > alpha): their groups adapt per token
    cfg = cfg_small(batch=2, n_kv_heads=2, n_q_heads=4, context=500, top_k=32, seed=42)
    st = Q2State(cfg, oracle, capacity=640, offset_std=1.0)
    dal, kvq = gpu_fit(st)
    rng = np.random.default_rng(0)
    K2, V2 = st.K.copy(), st.V.copy()
    new = W.make_cache(cfg, capacity=640, channel_offset_std=1.0, layer=3)
    K2[:, :, 500:633] = W.to_bits(W.from_bits(new[0][:, :, 500:633], cfg.dtype) * 3.0, cfg.dtype)
    V2[:, :, 500:633] = new[1][:, :, 500:633]
    qkv = oracle.quantize_kv(K2, V2, cfg.dtype, st.mu, st.alpha, 500, 133, st.qkv)
    codes = oracle.encode(K2, cfg.dtype, st.mu, 500, 133, st.codes)
    sik.sik_quantize_kv(st.layout, dev(K2, cfg.dtype), dev(V2, cfg.dtype), None, 500, 133, sik.SIK_Q_ENCODE, st.dmu,
                        dal, kvq)
    sync()
    got = kvq.cpu().numpy()
    check_records(st, got, K2, V2, qkv, codes, [(0, 0, 633), (1, 0, 633)], "encode range")
    assert not got[:, :, 633:].any()
    assert np.array_equal(dal.cpu().numpy(), st.alpha)      # frozen
    # empty range: nothing happens
    sik.sik_quantize_kv(st.layout, st.dK, st.dV, None, 10, 0, sik.SIK_Q_ENCODE, st.dmu, dal, kvq)
    sync()
    assert np.array_equal(kvq.cpu().numpy(), got)
    del rng


def test_degenerate_groups_and_channels(oracle):
    cfg = cfg_small(batch=1, n_kv_heads=2, n_q_heads=2, context=130, top_k=16, dtype="fp16", seed=43)
    K, V = W.make_cache(cfg)
    Kf, Vf = W.from_bits(K, "fp16").copy(), W.from_bits(V, "fp16").copy()
    Kf[0, 0, :, 5] = 0.75                    # a constant channel: K = mu there, alpha = 0
    Kf[0, 1, 7] = 0.0                        # a zero key row
    Vf[0, 0, 3] = 2.5                        # constant value row: qs = 0 in all four groups
    Vf[0, 1, 9, 32:64] = 0.0                 # an all-zero group
    Vf[0, 1, 11, 0:32] = np.where(np.arange(32) % 2 == 0, 0.0, -0.0)   # zeros of both signs only
    Vf[0, 1, 12, 0:32] = np.linspace(0, 3, 32)                         # exact ties at .5 do occur here
    K, V = W.to_bits(Kf, "fp16"), W.to_bits(Vf, "fp16")
    st = Q2State(cfg, oracle, K=K, V=V)
    assert st.alpha[0, 0, 5] == 0.0
    dal, kvq = gpu_fit(st)
    assert np.array_equal(dal.cpu().numpy(), st.alpha)
    got = kvq.cpu().numpy()
    check_records(st, got, K, V, st.qkv, st.codes, [(0, 0, 130)], "degenerate groups")
    # the planted groups are exact in any precision: constant row, zero group, zeros of both signs, the ramp with
    # its exact ties
    _, g = oracle.unpack_records(got)
    for (h, t, sl_) in ((0, 3, slice(0, 128)), (1, 9, slice(32, 64)), (1, 11, slice(0, 32)), (1, 12, slice(0, 32))):
        assert np.array_equal(g.vq[0, h, t, sl_], st.qkv.vq[0, h, t, sl_])
        gs = slice(sl_.start // 32, sl_.stop // 32)
        assert np.array_equal(g.vpar[0, h, t, gs], st.qkv.vpar[0, h, t, gs])
    assert not g.vpar[0, 0, 3, :, 0].any() and not g.vq[0, 0, 3].any()      # qs = 0 -> Q = 0
    assert not g.kq[0, 0, :, 5].any()        # dead channel: x = 0


@pytest.mark.parametrize("dtype,out_f32", [("bf16", True), ("fp16", True), ("bf16", False), ("fp16", False)])
def test_attention_on_records_matches_oracle(oracle, dtype, out_f32):
    cfg = cfg_small(batch=2, n_kv_heads=2, n_q_heads=8, context=3000, top_k=333, dtype=dtype, seed=44)
    st = Q2State(cfg, oracle, seq_len=[3000, 1777], offset_std=0.5, out_dtype=torch.float32 if out_f32 else None)
    kvq = torch.from_numpy(st.records()).cuda()
    dal = torch.from_numpy(st.alpha).cuda()
    q, _, _ = W.make_step_inputs(cfg, 0)
    idx = oracle.topk(oracle.score(q, dtype, st.cb, st.codes, st.sl), st.sl, 333)
    idx[0, 0, 5] = idx[0, 0, 6]              # a repeated entry counts twice
    idx[1, 3, 100:] = -1                     # padding is skipped
    out = torch.empty(2, 8, 128, dtype=torch.float32 if out_f32 else TDT[dtype], device="cuda")
    sik.sik_sparse_attn_q2(st.layout, dev(q, dtype), kvq, dal, torch.from_numpy(idx).cuda(), 333, 0.0, out, st.ws)
    sync()
    ref = oracle.sparse_attn_q2(q, dtype, st.codes, st.qkv, st.alpha, idx)
    check_attention(out.float().cpu().numpy().astype(np.float64), ref, out_f32, dtype)


def test_attention_on_records_all_tokens_and_small_selections(oracle):
    cfg = cfg_small(batch=1, n_kv_heads=2, n_q_heads=4, context=1100, top_k=1100, seed=45)
    st = Q2State(cfg, oracle, out_dtype=torch.float32)
    kvq = torch.from_numpy(st.records()).cuda()
    dal = torch.from_numpy(st.alpha).cuda()
    q, _, _ = W.make_step_inputs(cfg, 1)
    out = torch.empty(1, 4, 128, device="cuda")
    for k, idx in ((1100, np.tile(np.arange(1100, dtype=np.int32), (1, 4, 1))),
                   (1, np.full((1, 4, 1), 17, np.int32)),
                   (40, np.tile(np.arange(1060, 1100, dtype=np.int32)[::-1].copy(), (1, 4, 1))),
                   (5, np.full((1, 4, 5), -1, np.int32))):
        sik.sik_sparse_attn_q2(st.layout, dev(q, cfg.dtype), kvq, dal, torch.from_numpy(idx).cuda(), k, 0.09, out,
                               st.ws)
        sync()
        ref = oracle.sparse_attn_q2(q, cfg.dtype, st.codes, st.qkv, st.alpha, idx, scale=0.09)
        check_attention(out.cpu().numpy().astype(np.float64), ref, True)


# --------------------------------------------------------------------------- decode step on records
# launches = 1: the one-launch step on records whenever its plan allows (the library picks it for large launches only)
BOTH_PATHS = pytest.mark.parametrize("launches", [0, 1], ids=["auto", "one_launch"])


def run_decode_q2_and_check(oracle, cfg, capacity, steps, append, offset_std=0.0, seq_len=None, out_f32=True,
                            launches=0):
    st = Q2State(cfg, oracle, capacity=capacity, seq_len=seq_len, offset_std=offset_std,
                 out_dtype=torch.float32 if out_f32 else None)
    B, Hq, k = cfg.batch, cfg.n_q_heads, min(cfg.top_k, capacity)
    kvq = torch.from_numpy(st.records()).cuda()
    dal = torch.from_numpy(st.alpha).cuda()
    sl, codes, qkv = st.sl.copy(), st.codes, st.qkv
    out = torch.empty(B, Hq, 128, dtype=torch.float32 if out_f32 else TDT[cfg.dtype], device="cuda")
    idx = torch.empty(B, Hq, k, dtype=torch.int32, device="cuda")
    total_diff = 0
    for step in range(steps):
        q, kn, vn = W.make_step_inputs(cfg, step)
        dkn = dev(kn, cfg.dtype) if append else None
        dvn = dev(vn, cfg.dtype) if append else None
        if launches == 0:
            sik.sik_decode_step_q2(st.layout, dev(q, cfg.dtype), dkn, dvn, kvq, st.dsl, st.dmu, dal, st.dcb, st.dcodes,
                                   k, 0.0, out, idx, st.ws)
        else:
            sik.sik_decode_step_ex(st.layout, q=dev(q, cfg.dtype), k_new=dkn, v_new=dvn, kvq=kvq, alpha=dal,
                                   seq_len=st.dsl, mu=st.dmu, codebook=st.dcb, codes=st.dcodes, k=k, out=out,
                                   idx_out=idx, workspace=st.ws, launches=launches)
        sync()
        assert sik.sik_workspace_status(st.ws) == 0
        ref_out, ref_idx = oracle.decode_step_q2(q, kn if append else None, vn if append else None, cfg.dtype, sl,
                                                 st.mu, st.alpha, st.cb, codes, qkv, k)
        assert np.array_equal(st.dsl.cpu().numpy(), sl)
        if append:
            adopt_appended_records(oracle, kvq, kn, vn, cfg.dtype, st.mu, st.alpha, codes, qkv, sl)
            for b in range(B):
                t = int(sl[b]) - 1
                assert np.array_equal(st.dcodes[b, :, t].cpu().numpy(), codes[b, :, t])
        g_idx = idx.cpu().numpy()
        s_ref = oracle.score(q, cfg.dtype, st.cb, codes, sl)
        for b in range(B):
            for hq in range(Hq):
                total_diff += topk_sets_agree(g_idx[b, hq], ref_idx[b, hq], s_ref[b, hq], int(sl[b]), k)
        ref_on_gpu_set = oracle.sparse_attn_q2(q, cfg.dtype, codes, qkv, st.alpha, g_idx)
        check_attention(out.float().cpu().numpy().astype(np.float64), ref_on_gpu_set, out_f32, cfg.dtype)
    return total_diff


@BOTH_PATHS
def test_decode_q2_c1_full(oracle, launches):
    run_decode_q2_and_check(oracle, W.CONFIGS["C1"], capacity=4096, steps=2, append=False, launches=launches)


@BOTH_PATHS
def test_decode_q2_c1_16bit_out(oracle, launches):
    run_decode_q2_and_check(oracle, W.CONFIGS["C1"], capacity=4096, steps=1, append=False, out_f32=False, launches=launches)


@BOTH_PATHS
def test_decode_q2_c2_shape_reduced(oracle, launches):
    run_decode_q2_and_check(oracle, cfg_small("C2", context=8192, top_k=256), capacity=8192, steps=2, append=False,
                            offset_std=1.0, launches=launches)


@BOTH_PATHS
def test_decode_q2_c3_shape_reduced_with_append(oracle, launches):
    run_decode_q2_and_check(oracle, cfg_small("C3", context=9000, top_k=300), capacity=9004, steps=3, append=True,
                            offset_std=1.0, launches=launches)


@BOTH_PATHS
def test_decode_q2_c4_shape_reduced_ragged_batch(oracle, launches):
    run_decode_q2_and_check(oracle, cfg_small("C4", batch=4, context=2048, top_k=512), capacity=2050, steps=1,
                            append=True, seq_len=[2048, 1, 511, 700], launches=launches)


@BOTH_PATHS
def test_decode_q2_c5_shape_reduced_gqa8_fp16(oracle, launches):
    cfg = cfg_small("C5", batch=2, n_kv_heads=2, n_q_heads=16, context=6000, top_k=1536, dtype="fp16")
    run_decode_q2_and_check(oracle, cfg, capacity=6016, steps=3, append=True, launches=launches)


@BOTH_PATHS
def test_decode_q2_dense_selection_and_k_above_context(oracle, launches):
    run_decode_q2_and_check(oracle, cfg_small("C2", context=20000, top_k=20000), capacity=20000, steps=1, append=False, launches=launches)
    run_decode_q2_and_check(oracle, cfg_small("C2", n_kv_heads=2, n_q_heads=8, context=700, top_k=1024),
                            capacity=1100, steps=1, append=True, launches=launches)


@BOTH_PATHS
def test_decode_q2_empty_and_single_token_sequences(oracle, launches):
    cfg = cfg_small("C2", batch=3, n_kv_heads=2, n_q_heads=4, context=300, top_k=16)
    run_decode_q2_and_check(oracle, cfg, capacity=320, steps=2, append=True, seq_len=[0, 1, 300], launches=launches)


def test_decode_q2_graph_replay_and_profiled(oracle):
    cfg = cfg_small("C2", context=20000, top_k=600)
    st = Q2State(cfg, oracle, capacity=20008, out_dtype=torch.float32)
    kvq = torch.from_numpy(st.records()).cuda()
    dal = torch.from_numpy(st.alpha).cuda()
    q, kn, vn = W.make_step_inputs(cfg, 0)
    dq, dkn, dvn = dev(q, cfg.dtype), dev(kn, cfg.dtype), dev(vn, cfg.dtype)
    out = torch.empty(1, 32, 128, device="cuda")
    idx = torch.empty(1, 32, 600, dtype=torch.int32, device="cuda")

    def body(prof=False):
        st.dsl.fill_(20000)
        return sik.sik_decode_step_q2(st.layout, dq, dkn, dvn, kvq, st.dsl, st.dmu, dal, st.dcb, st.dcodes, 600, 0.0,
                                      out, idx, st.ws, profiled=prof)

    body()
    sync()
    eager_out, eager_idx = out.clone(), torch.sort(idx, dim=-1).values.clone()
    assert int(st.dsl[0]) == 20001
    us = body(prof=True)
    assert len(us) == 5 and us[1] > 0 and us[3] > 0 and torch.equal(out, eager_out)
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        body()
        sync()
        with torch.cuda.graph(g, stream=side):
            body()
    sync()
    for r in range(3):
        out.zero_()
        idx.fill_(-3)
        st.dsl.fill_(123)
        torch.randn(1 << 20, device="cuda").sum().item()
        g.replay()
        sync()
        assert int(st.dsl[0]) == 20001
        assert torch.equal(out, eager_out), r
        assert torch.equal(torch.sort(idx, dim=-1).values, eager_idx), r


@pytest.mark.parametrize("forced", [False, True])
def test_decode_q2_one_launch_graph_replay_with_append(oracle, forced):
    # the one-launch step on records (and with a forced set that names the appended token) under graph replay: its
    # counters are left at zero by every replay, the appended record and the published length are the eager ones
    cfg = cfg_small("C3", context=20000, top_k=600)
    st = Q2State(cfg, oracle, capacity=20008, out_dtype=torch.float32)
    kvq0 = torch.from_numpy(st.records()).cuda()
    kvq, dal = kvq0.clone(), torch.from_numpy(st.alpha).cuda()
    q, kn, vn = W.make_step_inputs(cfg, 0)
    dq, dkn, dvn = dev(q, cfg.dtype), dev(kn, cfg.dtype), dev(vn, cfg.dtype)
    out = torch.empty(1, 32, 128, device="cuda")
    idx = torch.empty(1, 32, 600, dtype=torch.int32, device="cuda")
    fidx = None
    if forced:
        f = np.tile(np.arange(0, 64 * 300, 300, dtype=np.int32), (1, 8, 1))
        f[:, :, 0] = 20000                       # the token being appended
        fidx = torch.from_numpy(f).cuda()

    def body(launches=1):
        st.dsl.fill_(20000)
        sik.sik_decode_step_ex(st.layout, q=dq, k_new=dkn, v_new=dvn, kvq=kvq, alpha=dal, seq_len=st.dsl, mu=st.dmu,
                               codebook=st.dcb, codes=st.dcodes, k=600, out=out, idx_out=idx, workspace=st.ws,
                               forced_idx=fidx, launches=launches)

    body(launches=2)
    sync()
    ref_out, ref_idx, ref_rec = out.clone(), torch.sort(idx, dim=-1).values.clone(), kvq[:, :, 20000].clone()
    kvq.copy_(kvq0)
    body()
    sync()
    assert sik.sik_workspace_status(st.ws) == 0 and int(st.dsl[0]) == 20001
    eager_out = out.clone()
    assert torch.equal(torch.sort(idx, dim=-1).values, ref_idx) and torch.equal(kvq[:, :, 20000], ref_rec)
    assert float((eager_out - ref_out).abs().max()) <= 2e-5 * float(ref_out.abs().max())
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        body()
        sync()
        with torch.cuda.graph(g, stream=side):
            body()
    sync()
    for r in range(3):
        out.zero_()
        idx.fill_(-3)
        kvq.copy_(kvq0)
        torch.randn(1 << 20, device="cuda").sum().item()
        g.replay()
        sync()
        assert sik.sik_workspace_status(st.ws) == 0 and int(st.dsl[0]) == 20001
        assert torch.equal(out, eager_out), r
        assert torch.equal(torch.sort(idx, dim=-1).values, ref_idx), r
        assert torch.equal(kvq[:, :, 20000], ref_rec), r


def test_decode_q2_rejects_contexts_without_a_fused_plan(oracle):
    lay = sik.make_layout(1, 1, 1, 128, 600000, torch.bfloat16, torch.float32)
    ws = sik.alloc_workspace(lay, 16)
    t = torch.zeros(16, device="cuda")
    with pytest.raises(sik.SikError) as e:
        sik.sik_decode_step_q2(lay, t, None, None, t, t, t, t, t, t, 16, 0.0, t, None, ws)
    assert e.value.status == -2


# --------------------------------------------------------------------------- prefill-compress in one call
@pytest.mark.parametrize("dtype,seq_len", [("bf16", [5000, 1337, 1, 0]), ("fp16", [4099, 4100, 777, 64])])
def test_prefill_compress_equals_the_separate_calls_and_the_oracle(oracle, dtype, seq_len):
    # one call, two passes over K and one over V: every output has the bits of sik_quantize_keys FIT followed by
    # sik_quantize_kv FIT, and agrees with the oracle as those do
    cfg = cfg_small(batch=4, n_kv_heads=3, n_q_heads=6, context=max(seq_len), top_k=64, dtype=dtype, seed=47)
    st = Q2State(cfg, oracle, capacity=max(seq_len) + 20, seq_len=seq_len, offset_std=1.2)
    B, H, cap = 4, 3, max(seq_len) + 20

    def fresh():
        return (torch.full((B, H, 128), -3.0, device="cuda"), torch.full((B, H, 32, 16, 4), -3.0, device="cuda"),
                torch.full((B, H, 32, 16), -3, dtype=torch.int32, device="cuda"),
                torch.zeros(B, H, cap, 16, dtype=torch.uint8, device="cuda"), torch.full((B, H, 128), -3.0, device="cuda"),
                sik.alloc_kvq(st.layout))

    mu1, cb1, cnt1, codes1, al1, rec1 = fresh()
    sik.sik_quantize_keys(st.layout, st.dK, st.dsl, 0, 0, sik.SIK_Q_FIT, mu1, cb1, cnt1, codes1, st.ws)
    sik.sik_quantize_kv(st.layout, st.dK, st.dV, st.dsl, 0, 0, sik.SIK_Q_FIT, mu1, al1, rec1)
    mu2, cb2, cnt2, codes2, al2, rec2 = fresh()
    sik.sik_prefill_compress(st.layout, st.dK, st.dV, st.dsl, mu2, cb2, cnt2, codes2, al2, rec2, st.ws)
    sync()
    for name, a, b in (("mu", mu1, mu2), ("codebook", cb1, cb2), ("counts", cnt1, cnt2), ("codes", codes1, codes2),
                       ("alpha", al1, al2), ("records", rec1, rec2)):
        assert torch.equal(a, b), name
    assert np.array_equal(mu2.cpu().numpy(), st.mu) and np.array_equal(al2.cpu().numpy(), st.alpha)
    assert np.array_equal(cnt2.cpu().numpy(), oracle.fit(st.K, dtype, st.sl)[3])
    got = rec2.cpu().numpy()
    check_records(st, got, st.K, st.V, st.qkv, st.codes, [(b, 0, int(L)) for b, L in enumerate(st.sl)],
                  f"prefill-compress {dtype}")
    for b, L in enumerate(st.sl):
        assert np.array_equal(codes2[b, :, :L].cpu().numpy(), st.codes[b, :, :L])
        assert not got[b, :, L:].any() and not codes2[b, :, L:].any()


@pytest.mark.parametrize("batch,lens", [(1, [16]), (1, [257]), (1, [513]), (5, [2048]), (5, [2049, 300]), (1, [16385]),
                                        (8, [5376]), (8, [5377, 65]), (40, [8195, 77]), (42, [8195, 8100, 0]),
                                        (43, [6145, 1, 5000])])
def test_fit_partials_and_slices(oracle, batch, lens):
    # 1 to 64 partials per unit (at least 256 rows each): one slice with two per thread (1, 2) or eight (3, 8), two slices
    # (9, 16: 42 x 3 units) and eight (17: 40 x 3 units, and more) in the reductions
    B, H, cap = batch, 3, max(lens)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(cap)
    lens = [lens[b % len(lens)] for b in range(B)]
    lay = sik.make_layout(B, H, 6, 128, cap, torch.bfloat16, torch.bfloat16)
    K, V = (torch.randn(B, H, cap, 128, generator=gen, device="cuda").add_(0.7).to(torch.bfloat16) for _ in range(2))
    dsl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    ws = sik.alloc_workspace(lay, 16)
    res = []
    for one_call in (False, True):
        mu, al = torch.zeros(B, H, 128, device="cuda"), torch.zeros(B, H, 128, device="cuda")
        cb = torch.zeros(B, H, 32, 16, 4, device="cuda")
        cnt = torch.zeros(B, H, 32, 16, dtype=torch.int32, device="cuda")
        codes, rec = torch.zeros(B, H, cap, 16, dtype=torch.uint8, device="cuda"), sik.alloc_kvq(lay)
        if one_call:
            sik.sik_prefill_compress(lay, K, V, dsl, mu, cb, cnt, codes, al, rec, ws)
        else:
            sik.sik_quantize_keys(lay, K, dsl, 0, 0, sik.SIK_Q_FIT, mu, cb, cnt, codes, ws)
            sik.sik_quantize_kv(lay, K, V, dsl, 0, 0, sik.SIK_Q_FIT, mu, al, rec)
        res.append((mu, cb, cnt, codes, al, rec))
    sync()
    for a, b in zip(*res):
        assert torch.equal(a, b)
    mu, cb, cnt, codes, al = (x.cpu().numpy() for x in res[0][:5])
    for b in {0, 1 % B, 2 % B, B - 1}:
        n = lens[b]
        x = K[b, :, :n].cpu().double().numpy()
        m = (x.sum(1) / n if n else np.zeros((H, 128))).astype(np.float32)
        assert np.array_equal(mu[b], m)
        peak = np.abs(x.astype(np.float32) - m[:, None]).max(1) if n else np.zeros((H, 128), np.float32)
        assert np.array_equal(al[b], peak)
        sign = x >= m[:, None]
        assert np.array_equal(codes[b, :, :n], np.packbits(sign, axis=-1))
        code = (sign.reshape(H, n, 32, 4) * [8, 4, 2, 1]).sum(-1)
        y = (x - m[:, None].astype(np.float64)).reshape(H, n, 32, 4)
        for c in range(16):
            hit = code == c
            want = hit.sum(1)
            assert np.array_equal(cnt[b, :, :, c], want)
            mean = (y * hit[..., None]).sum(1) / np.maximum(want, 1)[..., None]
            # binary32 sums of at most 2048 differences of one sign: each addition rounds by 2^-24 of the running sum
            peak = (np.abs(y) * hit[..., None]).sum(1) / np.maximum(want, 1)[..., None]
            assert (np.abs(cb[b, :, :, c] - mean) <= 2050 * 2.0 ** -24 * peak + 1e-30).all()


def fit_sums_reference(x, mu, nwg):
    """Cluster sums of one (sequence, KV head) in the library's order of additions, x [n, 128] the keys and mu [128] the
    means, both binary32: a workgroup's token range is walked by four chains (token mod 4) that add K - mu in binary32 in
    token order, the chains join as (0 + 1) + (2 + 3), the workgroups in binary64."""
    n = x.shape[0]
    code = ((x >= mu).reshape(n, 32, 4) * [8, 4, 2, 1]).sum(-1)
    y = (x - mu).reshape(n, 32, 1, 4)
    masked = np.where((code[:, :, None] == np.arange(16))[..., None], y, np.float32(0))
    chunk = -(-(-(-n // nwg)) // 4) * 4
    total = np.zeros((32, 16, 4))
    for start in range(0, n, chunk):
        end = min(n, start + chunk)
        c = [np.cumsum(masked[start + j:end:4], axis=0, dtype=np.float32)[-1] if start + j < end
             else np.zeros((32, 16, 4), np.float32) for j in range(4)]
        total += ((c[0] + c[1]) + (c[2] + c[3])).astype(np.float64)
    return total


@pytest.mark.parametrize("one_call", [False, True])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("units,n", [(1, 3), (3, 257), (2, 2055), (40, 1030)])
def test_codebook_bits_follow_from_the_stated_order_of_additions(units, n, dtype, one_call):
    # a codebook decides which tokens later steps select: it must not move by an ulp with the shape of a launch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(units * n)
    lay = sik.make_layout(1, units, units, 128, n, dtype, dtype)
    K, V = (torch.randn(1, units, n, 128, generator=gen, device="cuda").add_(0.3).to(dtype) for _ in range(2))
    dsl = torch.tensor([n], dtype=torch.int32, device="cuda")
    mu, al = torch.zeros(1, units, 128, device="cuda"), torch.zeros(1, units, 128, device="cuda")
    cb = torch.zeros(1, units, 32, 16, 4, device="cuda")
    cnt = torch.zeros(1, units, 32, 16, dtype=torch.int32, device="cuda")
    codes = torch.zeros(1, units, n, 16, dtype=torch.uint8, device="cuda")
    ws = sik.alloc_workspace(lay, 0)
    if one_call:
        sik.sik_prefill_compress(lay, K, V, dsl, mu, cb, cnt, codes, al, sik.alloc_kvq(lay), ws)
    else:
        sik.sik_quantize_keys(lay, K, dsl, 0, 0, sik.SIK_Q_FIT, mu, cb, cnt, codes, ws)
    sync()
    nwg = min(2048 // units, 64, -(-n // 256))
    for h in {0, units - 1}:
        m, c = mu[0, h].cpu().numpy(), cnt[0, h].cpu().numpy()
        s = fit_sums_reference(K[0, h].cpu().float().numpy(), m, nwg)
        want = np.where(c[..., None] > 0, s / np.maximum(c, 1)[..., None], 0.0).astype(np.float32)
        assert np.array_equal(cb[0, h].cpu().numpy(), want)


def test_prefill_compress_argument_errors():
    lay = sik.make_layout(1, 2, 4, 128, 512, torch.bfloat16)
    ws = sik.alloc_workspace(lay, 0)
    t = torch.zeros(16, device="cuda")
    with pytest.raises(sik.SikError) as e:
        sik.sik_prefill_compress(lay, t, None, t, t, t, t, t, t, t, ws)
    assert e.value.status == -1
    with pytest.raises(sik.SikError) as e:
        sik.sik_prefill_compress(lay, t, t, t, t, t, t, t, t, t, torch.zeros(256, dtype=torch.uint8, device="cuda"))
    assert e.value.status == -6


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 128, 191])
def test_tokens_of_one_code_are_added_in_token_order(n, dtype):
    # The encoder takes a lane's tokens in twos and lets the second add to the first one's sum where their codes agree:
    # here they always do (all keys but the first lie above the mean), at the edges of its blocks of 32 and 64.
    x = torch.rand(n, 128, generator=torch.Generator().manual_seed(n)).add_(1.0)
    x[0] = -100.0 - 2.0 * n
    lay = sik.make_layout(1, 1, 1, 128, n, dtype, dtype)
    K = x.to(dtype)[None, None].cuda()
    dsl = torch.tensor([n], dtype=torch.int32, device="cuda")
    for one_call in (False, True):
        mu, al = torch.zeros(1, 1, 128, device="cuda"), torch.zeros(1, 1, 128, device="cuda")
        cb = torch.zeros(1, 1, 32, 16, 4, device="cuda")
        cnt = torch.zeros(1, 1, 32, 16, dtype=torch.int32, device="cuda")
        codes = torch.zeros(1, 1, n, 16, dtype=torch.uint8, device="cuda")
        ws = sik.alloc_workspace(lay, 0)
        if one_call:
            sik.sik_prefill_compress(lay, K, K, dsl, mu, cb, cnt, codes, al, sik.alloc_kvq(lay), ws)
        else:
            sik.sik_quantize_keys(lay, K, dsl, 0, 0, sik.SIK_Q_FIT, mu, cb, cnt, codes, ws)
        sync()
        m, k = mu[0, 0].cpu().numpy(), K[0, 0].cpu().float().numpy()
        assert (k[1:] >= m).all()
        assert np.array_equal(codes[0, 0].cpu().numpy(), np.packbits(k >= m, axis=-1))
        c = cnt[0, 0].cpu().numpy()
        assert c.sum() == 32 * n
        s = fit_sums_reference(k, m, 1)
        want = np.where(c[..., None] > 0, s / np.maximum(c, 1)[..., None], 0.0).astype(np.float32)
        assert np.array_equal(cb[0, 0].cpu().numpy(), want)


def check_groups(x, bits, par):
    """Records of groups x [n, 4, 32] (binary32, as the builder sees them) against the quantisation function: bits
    [n, 4, 4] the code words of a group's four lanes, par [n, 4, 2] its step and zero point.  A NaN among the values is
    left out of the extremes and has the code zero."""
    with np.errstate(all="ignore"):
        lo, hi = np.fmin.reduce(x, -1) + np.float32(0), np.fmax.reduce(x, -1)   # a zero minimum is +0
        zp = lo.astype(np.float16)
        # a zero step is +0; a span beyond binary32 has no third
        qs = np.where(np.isinf(hi - lo), np.float32(np.nan), (hi - lo) / np.float32(3) + np.float32(0)).astype(np.float16)
        for got, want in ((par[..., 0], qs), (par[..., 1], zp)):
            assert np.array_equal(np.isnan(got), np.isnan(want))
            assert np.array_equal(got.view(np.uint16)[~np.isnan(want)], want.view(np.uint16)[~np.isnan(want)])
        q = ((bits[..., None] >> (2 * np.arange(8, dtype=np.uint16))) & 3).reshape(x.shape)
        step = (qs > 0) & np.isfinite(qs)
        assert not q[~step].any()          # no step, or none that is a number: every code is zero
        assert not q[np.isnan(x)].any()
        t = (x - zp.astype(np.float32)[..., None]) / qs.astype(np.float32)[..., None]
        want = np.clip(np.rint((x - zp.astype(np.float32)[..., None])
                               * (np.float32(1) / qs.astype(np.float32))[..., None]), 0, 3)
        # (the factor is the reciprocal up to its last place: a quotient that close to a half may go either way)
        clear = (step & np.isfinite(zp))[..., None] & ~np.isnan(x) & (np.abs(t - np.floor(t) - 0.5) > 1e-6)
    assert np.array_equal(q[clear], want[clear])


def test_records_of_degenerate_groups_in_16_bits():
    # groups without a step, with extremes beyond binary16 or binary32, and with NaN, at every place of a quad's lanes
    gen = torch.Generator().manual_seed(5)
    n = 48
    V = torch.randn(1, 1, n, 128, generator=gen)
    V[0, 0, 1] = 0.0
    V[0, 0, 2, 32:64] = -0.0
    V[0, 0, 3] = 7.0
    V[0, 0, 4, 5] = 3.0e38        # the step is infinite
    V[0, 0, 5, 33] = -3.0e38
    V[0, 0, 6] = 1.0e38           # a constant whose zero point is infinite and whose step is zero
    for lane in range(4):         # an extreme held by each of the four lanes, and a value that is none
        V[0, 0, 8 + lane, 8 * lane] = 50.0
        V[0, 0, 12 + lane, 8 * lane + 7] = -50.0
        V[0, 0, 16 + lane, 8 * lane + lane] = float("nan")
        V[0, 0, 20 + lane, 32 + 8 * lane:40 + 8 * lane] = float("nan")  # all eight of a lane
    V[0, 0, 24, 64:96] = float("nan")
    V[0, 0, 25, 3], V[0, 0, 25, 30] = 3.0e38, -3.0e38  # their difference overflows: the step is NaN
    V[0, 0, 26, 100] = float("inf")
    V[0, 0, 27, 100] = float("-inf")
    V = V.to(torch.bfloat16)
    V.view(torch.int16)[0, 0, 28, 8] = 0x7f81          # a signalling NaN
    K = torch.randn(1, 1, n, 128, generator=gen).to(torch.bfloat16)
    K[0, 0, :, 32:64] = 0.75      # a group of channels that never leave their mean
    K[0, 0, 7, 70] = float("nan")  # its channel has no mean and no scale
    K[0, 0, 9, 96:104] = 40.0
    K, V = K.cuda(), V.cuda()
    lay = sik.make_layout(1, 1, 1, 128, n, torch.bfloat16, torch.bfloat16)
    dsl = torch.tensor([n], dtype=torch.int32, device="cuda")
    mu, al = torch.zeros(1, 1, 128, device="cuda"), torch.zeros(1, 1, 128, device="cuda")
    cb = torch.zeros(1, 1, 32, 16, 4, device="cuda")
    cnt = torch.zeros(1, 1, 32, 16, dtype=torch.int32, device="cuda")
    codes = torch.zeros(1, 1, n, 16, dtype=torch.uint8, device="cuda")
    kvq = sik.alloc_kvq(lay)
    sik.sik_prefill_compress(lay, K, V, dsl, mu, cb, cnt, codes, al, kvq, sik.alloc_workspace(lay, 0))
    sync()
    slots = kvq.cpu().numpy().reshape(n, 4, 4, 8)                  # token, group, lane of the quad, bytes
    kbits, vbits = (slots[..., a:a + 2].copy().view(np.uint16).reshape(n, 4, 4) for a in (2, 4))
    par = slots[..., 6:8].copy().view(np.float16).reshape(n, 4, 4)
    m, a = mu[0, 0].cpu().numpy(), al[0, 0].cpu().numpy()
    assert np.isnan(m[70]) and np.isfinite(np.delete(m, 70)).all() and not a[32:64].any()
    with np.errstate(all="ignore"):
        x = np.abs(K[0, 0].cpu().float().numpy() - m) * np.where(a > 0, np.float32(1) / a, np.float32(0))
    check_groups(x.reshape(n, 4, 32), kbits, par[..., 0:2])
    check_groups(V[0, 0].cpu().float().numpy().reshape(n, 4, 32), vbits, par[..., 2:4])


def test_attention_over_few_records_with_gaps(oracle):
    # two records are unpacked side by side: the first, the second or both of a pair missing, up to one gather step
    cfg = cfg_small(batch=1, n_kv_heads=1, n_q_heads=33, context=40, top_k=33, seed=46)
    st = Q2State(cfg, oracle, out_dtype=torch.float32)
    q, _, _ = W.make_step_inputs(cfg, 1)
    idx = np.full((1, 33, 33), -1, np.int32)
    rng = np.random.default_rng(46)
    for h in range(33):  # head h attends h + 1 records at places of the list drawn at random
        idx[0, h, rng.permutation(33)[:h + 1]] = rng.permutation(40)[:h + 1]
    out = torch.empty(1, 33, 128, device="cuda")
    sik.sik_sparse_attn_q2(st.layout, dev(q, cfg.dtype), torch.from_numpy(st.records()).cuda(),
                           torch.from_numpy(st.alpha).cuda(), torch.from_numpy(idx).cuda(), 33, 0.0, out, st.ws)
    sync()
    ref = oracle.sparse_attn_q2(q, cfg.dtype, st.codes, st.qkv, st.alpha, idx)
    check_attention(out.cpu().numpy().astype(np.float64), ref, True)
