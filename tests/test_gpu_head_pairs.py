"""The one-launch step with two heads to a workgroup (chunks of 8192 tokens and more on 16-bit rows), and the launch
structure that the library takes by itself: the tokens selected, and the attention over them, against the two-launch step
on the same cache, which shares none of the kernels."""
import numpy as np
import pytest
import torch

import paper_2603_14224_amd as sik

pytestmark = pytest.mark.gpu
TDT = {"bf16": torch.bfloat16, "fp16": torch.float16}


def build(B, Hkv, Hq, capacity, lens, k, dtype, seed, q2=False):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    lay = sik.make_layout(B, Hkv, Hq, 128, capacity, TDT[dtype], torch.float32)
    s = dict(lay=lay, ws=sik.alloc_workspace(lay, k), lens=torch.tensor(lens, dtype=torch.int32, device="cuda"))
    s["K"], s["V"] = (torch.randn(B, Hkv, capacity, 128, generator=gen, device="cuda", dtype=torch.float32).to(TDT[dtype])
                      for _ in range(2))
    s["mu"] = torch.empty(B, Hkv, 128, device="cuda")
    s["cb"] = torch.empty(B, Hkv, 32, 16, 4, device="cuda")
    s["codes"] = torch.zeros(B, Hkv, capacity, 16, dtype=torch.uint8, device="cuda")
    counts = torch.empty(B, Hkv, 32, 16, dtype=torch.int32, device="cuda")
    if q2:
        s["kvq"], s["alpha"] = sik.alloc_kvq(lay), torch.empty(B, Hkv, 128, device="cuda")
        sik.sik_prefill_compress(lay, s["K"], s["V"], s["lens"], s["mu"], s["cb"], counts, s["codes"], s["alpha"], s["kvq"],
                                 s["ws"])
    else:
        sik.sik_quantize_keys(lay, s["K"], s["lens"], 0, 0, sik.SIK_Q_FIT, s["mu"], s["cb"], counts, s["codes"], s["ws"])
    s["q"] = torch.randn(B, Hq, 128, generator=gen, device="cuda").to(TDT[dtype])
    s["new"] = [torch.randn(B, Hkv, 128, generator=gen, device="cuda").to(TDT[dtype]) for _ in range(2)]
    return s


def step(s, k, launches, append, q, per_mille=0, forced=None):
    lens, codes = s["lens"].clone(), s["codes"].clone()
    if "kvq" in s:
        kvq, K, V = s["kvq"].clone(), None, None
    else:
        kvq, (K, V) = None, ((s["K"].clone(), s["V"].clone()) if append else (s["K"], s["V"]))
    B, Hq = q.shape[:2]
    out = torch.full((B, Hq, 128), np.nan, device="cuda")
    idx = torch.full((B, Hq, k), -7, dtype=torch.int32, device="cuda")
    sik.sik_decode_step_ex(s["lay"], q=q, k_new=s["new"][0] if append else None, v_new=s["new"][1] if append else None, K=K,
                           V=V, kvq=kvq, alpha=s.get("alpha"), forced_idx=forced, seq_len=lens, mu=s["mu"], codebook=s["cb"], codes=codes, k=k, k_per_mille=per_mille,
                           out=out, idx_out=idx, workspace=s["ws"], launches=launches)
    torch.cuda.synchronize()
    assert sik.sik_workspace_status(s["ws"]) == 0
    return out, torch.sort(idx, dim=-1).values, lens, codes, *((K, V) if kvq is None else (kvq,))


# tokens of a chunk: 8192, 12288, 16384, 18432, 20480; heads of a group: whole and half pairs; one and several chunks
CASES = [
    (33, 8, 24, 8192, 256, "bf16", False),    # one chunk of 8192, more workgroups than two per compute unit, 2 + 1 heads
    (32, 8, 16, 8200, 100, "fp16", True),     # one chunk of 12288 mostly empty, one pair per KV head
    (16, 8, 40, 12289, 617, "bf16", True),    # one chunk of 16384, 2 + 2 + 1 heads
    (16, 8, 56, 18000, 700, "fp16", False),   # 2 + 2 + 2 + 1 heads
    (16, 8, 32, 36864, 1500, "bf16", True),   # two chunks of 18432, the second one full
    (16, 8, 32, 36866, 4, "fp16", True),      # two chunks of 20480
    (10, 8, 40, 24000, 900, "bf16", True),    # two chunks of 12288, more head blocks of four than half the compute units
]


@pytest.mark.parametrize("B,Hkv,Hq,L,k,dtype,append", CASES)
def test_head_pairs_pick_what_two_launches_pick(B, Hkv, Hq, L, k, dtype, append):
    lens = [max(0, L - append - (b * 977 if b % 3 else 0)) for b in range(B)]
    lens[1:5] = [0, 1, k, 8191]
    s = build(B, Hkv, Hq, L, lens, k, dtype, seed=L)
    tokens = sik.sik_plan_info(s["lay"])[7] * 1024
    assert tokens >= 8192
    for q in (s["q"], torch.zeros_like(s["q"])):  # zero: all scores equal, the threshold bin holds every token
        want = step(s, k, 2, append, q)
        got = step(s, k, 1, append, q)
        for a, b in zip(got[1:], want[1:]):
            assert torch.equal(a, b)
        # binary32 sums over the same rows in another order (chunk and slice sizes differ)
        scale = want[0].abs().amax(dim=-1, keepdim=True)
        assert bool(((got[0] - want[0]).abs() <= 2e-5 * scale).all())
        again = step(s, k, 1, append, q)
        assert torch.equal(again[0], got[0])  # the same bits whatever the order of arrival


def test_head_pairs_budget_follows_the_context():
    s = build(16, 8, 32, 16384, [16384 - 700 * b for b in range(16)], 1229, "bf16", seed=3)
    want, got = (step(s, 1229, launches, False, s["q"], per_mille=75) for launches in (2, 1))
    assert torch.equal(got[1], want[1])
    assert bool(((got[0] - want[0]).abs() <= 2e-5 * want[0].abs().amax(dim=-1, keepdim=True)).all())


# around the lines between the routes: contexts at and beyond the chunk sizes, few and many head blocks, several rounds
@pytest.mark.parametrize("forced", [0, 32], ids=["plain", "forced"])
@pytest.mark.parametrize("q2", [False, True], ids=["rows", "records"])
@pytest.mark.parametrize("B,Hkv,Hq,L,k", [(1, 1, 4, 1024, 60), (1, 1, 4, 1025, 60), (3, 2, 6, 2048, 100), (3, 2, 6, 2049, 100),
                                          (10, 8, 32, 4096, 2000), (20, 8, 32, 4097, 170), (8, 8, 32, 8192, 333),
                                          (5, 8, 40, 12288, 500), (20, 4, 28, 20480, 700), (48, 8, 16, 1000, 33),
                                          (34, 8, 64, 1030, 50)])
def test_route_taken_by_itself(B, Hkv, Hq, L, k, q2, forced):
    lens = [max(0, L - 1 - (b * 131 if b % 2 else 0)) for b in range(B)]
    s = build(B, Hkv, Hq, L, lens, k, "bf16", seed=L + B, q2=q2)
    # forced tokens anywhere in the longest sequence, some of them beyond the end of a shorter one
    named = torch.randint(0, L, (B, Hkv, forced), device="cuda", dtype=torch.int32).sort(-1).values if forced else None
    if forced:
        named[..., 1:][named[..., 1:] == named[..., :-1]] = -1  # a token is named once
    want, got = (step(s, k, launches, True, s["q"], forced=named) for launches in (2, 0))
    for a, b in zip(got[1:], want[1:]):
        assert torch.equal(a, b)
    assert bool(((got[0] - want[0]).abs() <= 2e-5 * want[0].abs().amax(dim=-1, keepdim=True)).all())


# (batch, KV heads, query heads, capacity, records, forced tokens, one launch?), both sides of the lines of step_single_pays
ROUTES = [(1, 1, 4, 1024, False, 0, True), (1, 1, 4, 2049, False, 0, False), (8, 8, 16, 8192, False, 0, False),
          (10, 8, 16, 8192, False, 0, True), (9, 4, 36, 8192, False, 0, True), (33, 8, 32, 2000, False, 0, False),
          (46, 8, 32, 2000, False, 0, True), (41, 8, 40, 4096, False, 0, False),
          (16, 8, 16, 20000, False, 0, True), (12, 8, 16, 20000, False, 0, False), (27, 8, 40, 10922, True, 0, True),
          (52, 8, 16, 9500, True, 0, True), (24, 8, 40, 16384, True, 0, False), (17, 8, 40, 8192, True, 0, False),
          (18, 8, 32, 16384, True, 0, True), (9, 8, 40, 16384, True, 0, False), (6, 8, 40, 4096, True, 64, False),
          (6, 8, 40, 3000, True, 64, True), (17, 8, 40, 16384, False, 64, False), (32, 8, 64, 8192, False, 64, True),
          (24, 8, 40, 8192, False, 64, False), (10, 8, 40, 24000, False, 0, True), (10, 8, 40, 28809, True, 0, False)]


@pytest.mark.parametrize("B,Hkv,Hq,capacity,q2,forced,one", ROUTES)
def test_launches_taken_by_itself(B, Hkv, Hq, capacity, q2, forced, one):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lines are drawn for 256 compute units")
    lay = sik.make_layout(B, Hkv, Hq, 128, capacity, torch.bfloat16, torch.float32)
    k = 32 + forced
    rows = dict(K=None, V=None, kvq=sik.alloc_kvq(lay), alpha=torch.ones(B, Hkv, 128, device="cuda")) if q2 else \
        {n: torch.zeros(B, Hkv, capacity, 128, device="cuda", dtype=torch.bfloat16) for n in "KV"}
    us = sik.sik_decode_step_ex(
        lay, q=torch.zeros(B, Hq, 128, device="cuda", dtype=torch.bfloat16), **rows, mu=torch.zeros(B, Hkv, 128, device="cuda"),
        seq_len=torch.full((B,), 200, dtype=torch.int32, device="cuda"), codebook=torch.zeros(B, Hkv, 32, 16, 4, device="cuda"),
        codes=torch.zeros(B, Hkv, capacity, 16, dtype=torch.uint8, device="cuda"), k=k,
        forced_idx=torch.arange(forced, dtype=torch.int32, device="cuda").repeat(B, Hkv, 1) if forced else None,
        out=torch.empty(B, Hq, 128, device="cuda"), workspace=sik.alloc_workspace(lay, k), profiled=True)
    assert (us[1] == 0.0) == one and us[3] > 0.0


def test_one_workspace_for_layouts_of_different_size():
    # initialised for the small layout only: what its launches leave behind its own counters must not meet the larger
    # layout's, whose appends are counted there
    small = build(1, 1, 4, 3000, [2990], 64, "bf16", seed=1)
    large = build(20, 8, 32, 4000, [3990 - b for b in range(20)], 64, "bf16", seed=2)
    shared = torch.randint(1, 255, (large["ws"].numel(),), dtype=torch.uint8, device="cuda")
    sik.sik_workspace_init(small["lay"], 64, shared)
    want = [step(s, 64, 2, True, s["q"]) for s in (small, large)]
    small["ws"] = large["ws"] = shared
    for _ in range(2):
        for s, w in zip((small, large), want):
            got = step(s, 64, 0, True, s["q"])
            assert all(torch.equal(a, b) for a, b in zip(got[1:], w[1:]))


def test_one_workspace_beyond_the_reserved_counters():
    # 16640 query-head rows need more counters than every workspace keeps: the last of them lie where the small layout
    # keeps its histograms
    small = build(1, 8, 32, 4096, [4090], 8, "bf16", seed=1)
    large = build(520, 8, 32, 64, [63 - b % 60 for b in range(520)], 8, "bf16", seed=2)
    want = [step(s, 8, 2, True, s["q"]) for s in (small, large)]
    sik.sik_workspace_init(large["lay"], 8, large["ws"])
    small["ws"] = large["ws"]
    for _ in range(2):
        for s, w in zip((small, large), want):
            got = step(s, 8, 0, True, s["q"])
            assert all(torch.equal(a, b) for a, b in zip(got[1:], w[1:]))


# lengths on both sides of the candidates that a workgroup of its own ranks (512) and that anything ranks (1024)
@pytest.mark.parametrize("forced", [0, 8], ids=["plain", "forced"])
@pytest.mark.parametrize("Hq,capacity,q2", [(8, 2048, False), (10, 2048, True), (6, 9000, False)])
def test_equal_scores_around_the_ranking_limits(Hq, capacity, q2, forced):
    lens = [n + d + forced for n in (512, 1024) for d in (-9, -1, 0, 1, 9)]
    s = build(len(lens), 2, Hq, capacity, lens, 100, "bf16", seed=Hq, q2=q2)
    named = (2 * torch.arange(forced, device="cuda", dtype=torch.int32)).repeat(len(lens), 2, 1).contiguous() if forced else None
    q = torch.zeros_like(s["q"])
    want, got, again = (step(s, 100, n, False, q, forced=named) for n in (2, 1, 1))
    assert torch.equal(got[1], want[1]) and torch.equal(got[0], again[0])
    assert bool(((got[0] - want[0]).abs() <= 2e-5 * want[0].abs().amax(dim=-1, keepdim=True)).all())


# every one-launch variant: one chunk of 2048, a pair's chunk of 16384, two chunks, records, the 16-bit first pass
@pytest.mark.parametrize("forced", [0, 16], ids=["plain", "forced"])
@pytest.mark.parametrize("B,Hkv,Hq,L,q2,launches", [(3, 2, 8, 2000, False, 1), (12, 8, 40, 15000, False, 1),
                                                    (2, 8, 32, 30000, False, 1), (3, 2, 6, 3000, True, 1),
                                                    (3, 2, 8, 4000, False, 3)])
def test_query_that_is_not_finite(B, Hkv, Hq, L, q2, launches, forced):
    # scores that are infinite or not numbers all lie in one bin, with more members than are ranked: the tokens taken are
    # those of the two-launch step, and no slot of the index rows is left as it was
    s = build(B, Hkv, Hq, L, [L] * B, L - 1, "bf16", seed=L, q2=q2)
    named = (3 * torch.arange(forced, device="cuda", dtype=torch.int32)).repeat(B, Hkv, 1).contiguous() if forced else None
    for h, x in enumerate((float("nan"), float("inf"), float("-inf"))):
        s["q"][:, h, 7] = x
    # (the two launches give a forced token the score -inf: at most its match among the scores, and above the negative NaNs
    # of scores that overflow, so those two are compared without forced tokens only)
    if not forced:
        s["q"][:, 3] = 3e38
    for k in (300,) if forced else (300, min(L - 1, 2500)):
        want, got = (step(s, k, n, False, s["q"], forced=named) for n in (2, launches))
        assert torch.equal(got[1], want[1]) and int(got[1].min()) >= -1
        bad = 3 if forced else 4
        assert torch.equal(got[0][:, :bad], want[0][:, :bad])  # no number comes out of these rows: zero either way


@pytest.mark.parametrize("launches,forced", [(1, 16), (3, 0)], ids=["forced", "first pass of 16 bits"])
def test_scores_with_the_bits_of_a_token_that_does_not_compete(launches, forced):
    # every score is the NaN that marks such tokens: all are equal, so the lowest indices are taken, forced ones first
    s = build(3, 2, 8, 4000, [4000, 3999, 1025 + forced], 300, "bf16", seed=11)
    s["cb"].view(torch.int32).fill_(-1)
    named = (3 * torch.arange(forced, device="cuda", dtype=torch.int32)).repeat(3, 2, 1).contiguous() if forced else None
    got = step(s, 300, launches, False, s["q"], forced=named)
    taken = set(range(0, 3 * forced, 3))
    want = sorted(taken) + [i for i in range(300 + forced) if i not in taken][:300 - forced]
    assert torch.equal(got[1], torch.tensor(sorted(want), dtype=torch.int32, device="cuda").expand_as(got[1]))
