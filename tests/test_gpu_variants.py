"""GPU parity of the path's variants (through the C ABI) against the fp64 oracle.

Grouped-query heads (prefill and decode), bf16 output, the row log-sum-exp,
a caller-provided decode workspace, and prefill with split key ranges.  Inputs are seeded bf16 N(0,1).
Tolerances: outputs as the main parity tests (max-abs 2e-2, mean-abs 2e-3);
the log-sum-exp within 5e-3 (the kernel's normaliser sums bf16-rounded
probabilities, each within a relative 2^-8 of its exact value, so log l is
within 2^-8 = 3.9e-3 of exact, plus fp32 accumulation of the scores).
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import pytest
import torch

import oracle
from attn_inputs import random_bf16
from tests.gpu_common import announce, compare, forced_plan

pytestmark = pytest.mark.gpu

DEV = "cuda"
LSE_MAX_ABS = 5e-3
LSE_MEAN_ABS = 1e-3


@pytest.fixture(scope="module")
def pa():
    import paper_2609_29219_amd as pa
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return pa


def _qkv(B, Hq, Hkv, Sq, Skv, d, seed):
    return (random_bf16((B, Hq, Sq, d), seed), random_bf16((B, Hkv, Skv, d), seed + 1),
            random_bf16((B, Hkv, Skv, d), seed + 2))


GQA_SHAPES = [  # B, Hq, Hkv, Sq, Skv, d, causal
    (2, 4, 2, 77, 130, 128, False),
    (1, 8, 2, 200, 200, 128, True),
    (1, 6, 1, 65, 300, 64, False),
    (2, 8, 8, 130, 130, 64, True),
    (1, 16, 2, 33, 257, 128, True),
]


@pytest.mark.parametrize("shape", GQA_SHAPES, ids=[str(s) for s in GQA_SHAPES])
def test_fwd_gqa_lse(pa, shape):
    B, Hq, Hkv, Sq, Skv, d, causal = shape
    q, k, v = _qkv(B, Hq, Hkv, Sq, Skv, d, 700 + Hq + Sq)
    sc = float(np.float32(1.0 / math.sqrt(d)))
    announce(f"attn_fwd_ex gqa {shape}")
    o, lse = pa.attn_fwd(q.to(DEV), k.to(DEV), v.to(DEV), scale=sc, causal=causal,
                         return_lse=True)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.attn_gqa(q, k, v, B, Hq, Hkv, Sq, Skv, d, sc, causal)
    compare(o, ref, f"gqa out {shape}")
    compare(lse, ref_lse, f"gqa lse {shape}", max_abs=LSE_MAX_ABS, mean_abs=LSE_MEAN_ABS)


@pytest.mark.parametrize("variant", [(64, 8, 1), (128, 8, 1), (64, 4, 0), (64, 8, 2), (64, 8, 3),
                                     (32, 4, 3)])
def test_fwd_gqa_every_schedule(pa, variant):
    B, Hq, Hkv, Sq, Skv, d = 1, 8, 2, 290, 290, 128
    q, k, v = _qkv(B, Hq, Hkv, Sq, Skv, d, 800)
    sc = float(np.float32(1.0 / math.sqrt(d)))
    with forced_plan(*variant):
        for causal in (False, True):
            announce(f"attn_fwd_ex gqa variant {variant} causal={causal}")
            o, lse = pa.attn_fwd(q.to(DEV), k.to(DEV), v.to(DEV), scale=sc, causal=causal,
                                 return_lse=True)
            torch.cuda.synchronize()
            ref, ref_lse = oracle.attn_gqa(q, k, v, B, Hq, Hkv, Sq, Skv, d, sc, causal)
            compare(o, ref, f"variant {variant}")
            compare(lse, ref_lse, f"variant {variant} lse", max_abs=LSE_MAX_ABS,
                    mean_abs=LSE_MEAN_ABS)


@pytest.mark.parametrize("causal", [False, True])
def test_fwd_bf16_output_is_the_rounded_fp32_output(pa, causal):
    B, H, Sq, Skv, d = 2, 3, 150, 150, 128
    q, k, v = _qkv(B, H, H, Sq, Skv, d, 900)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    announce(f"attn_fwd_ex bf16 output causal={causal}")
    o32 = pa.attn_fwd(qd, kd, vd, causal=causal)
    o16 = pa.attn_fwd(qd, kd, vd, causal=causal, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    assert o16.dtype == torch.bfloat16
    # same arithmetic, then round to nearest even: bit-exact
    assert torch.equal(o16.cpu(), o32.cpu().to(torch.bfloat16))
    ref = oracle.attn(q, k, v, B, H, Sq, Skv, d, float(np.float32(1 / math.sqrt(d))), causal)
    compare(o16.float(), ref, "bf16 output")


CAUSAL_SCHEDULES = [(32, 4, 0), (32, 8, 1), (64, 4, 1), (64, 8, 1), (32, 4, 3), (64, 8, 3),
                    (128, 8, 0), (64, 8, 2)]


@pytest.mark.parametrize("variant", CAUSAL_SCHEDULES, ids=[str(v) for v in CAUSAL_SCHEDULES])
@pytest.mark.parametrize("d", [64, 128])
def test_fwd_causal_rows_stored_early_every_schedule(pa, variant, d):
    # A causal wave whose last key tile comes before its q-tile's last one
    # stores its rows straight from registers while the other waves still
    # compute.  Ragged Sq < Skv (the diagonal is offset), and several q-tiles
    # so that workgroups run two passes; fp32 and bf16 rows and the LSE.
    B, H, Sq, Skv = 1, 3, 600, 633
    q, k, v = _qkv(B, H, H, Sq, Skv, d, 950 + d)
    sc = float(np.float32(1.0 / math.sqrt(d)))
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    with forced_plan(*variant):
        announce(f"attn_fwd_ex causal early stores {variant} d={d}")
        o, lse = pa.attn_fwd(qd, kd, vd, scale=sc, causal=True, return_lse=True)
        o16 = pa.attn_fwd(qd, kd, vd, scale=sc, causal=True, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.attn_gqa(q, k, v, B, H, H, Sq, Skv, d, sc, True)
    compare(o, ref, f"causal {variant} d={d}")
    compare(lse, ref_lse, f"causal {variant} d={d} lse", max_abs=LSE_MAX_ABS,
            mean_abs=LSE_MEAN_ABS)
    assert torch.equal(o16.cpu(), o.cpu().to(torch.bfloat16))


def test_fwd_lse_special_cases(pa):
    # Q = 0: every allowed score is 0, lse = log(#allowed keys) (exact up to fp32)
    B, H, Sq, Skv, d = 1, 2, 100, 160, 64
    k, v = random_bf16((B, H, Skv, d), 950), random_bf16((B, H, Skv, d), 951)
    q0 = torch.zeros((B, H, Sq, d), dtype=torch.bfloat16)
    announce("attn_fwd_ex lse with Q = 0")
    for causal in (False, True):
        _, lse = pa.attn_fwd(q0.to(DEV), k.to(DEV), v.to(DEV), causal=causal, return_lse=True)
        torch.cuda.synchronize()
        n = np.full(Sq, Skv) if not causal else np.arange(Sq) + (Skv - Sq) + 1
        np.testing.assert_allclose(lse.cpu().double().numpy(),
                                   np.broadcast_to(np.log(n), (B, H, Sq)), atol=2e-6, rtol=0)


def test_fwd_ex_rejects_before_launch(pa):
    q = torch.zeros((1, 4, 8, 64), dtype=torch.bfloat16, device=DEV)
    k = torch.zeros((1, 3, 8, 64), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(pa.AttnError) as e:
        pa.attn_fwd(q, k, k)  # 3 key/value heads do not divide 4 query heads
    assert e.value.code == pa.ATTN_EINVAL


DECODE_GQA = [  # B, Hq, Hkv, Skv, d, n_splits  (group >= 4: the matrix-core kernel)
    (2, 8, 2, 1000, 128, 0),
    (1, 32, 4, 4096, 128, 0),
    (3, 6, 2, 777, 64, 5),
    (1, 16, 1, 2049, 128, 0),
    (2, 12, 4, 300, 128, 3),
    (1, 32, 2, 8192, 64, 0),
    (2, 32, 1, 1500, 128, 0),   # MQA: two query blocks of 16
    (1, 48, 2, 700, 128, 4),    # group 24: a full and a partial query block
    (3, 8, 2, 33, 128, 0),      # fewer keys than one 32-key step per wave
    (2, 20, 4, 1, 64, 0),       # a single key
    (1, 64, 8, 65536, 128, 0),  # long context, group 8
    (2, 8, 2, 1000, 128, 1),    # one split: the matrix-core kernel writes o and lse itself
    (3, 6, 2, 777, 64, 1),      # one split, the VALU kernel (group 3)
]


@pytest.mark.parametrize("shape", DECODE_GQA, ids=[str(s) for s in DECODE_GQA])
def test_decode_gqa_lse(pa, shape):
    B, Hq, Hkv, Skv, d, n = shape
    q = random_bf16((B, Hq, d), 1000 + Hq)
    k, v = random_bf16((B, Hkv, Skv, d), 1001 + Hq), random_bf16((B, Hkv, Skv, d), 1002 + Hq)
    announce(f"attn_decode_ex gqa {shape}")
    o, lse = pa.attn_decode(q.to(DEV), k.to(DEV), v.to(DEV), n_splits=n, return_lse=True)
    torch.cuda.synchronize()
    sc = float(np.float32(1.0 / math.sqrt(d)))
    ref, ref_lse = oracle.attn_gqa(q.reshape(B, Hq, 1, d).contiguous(), k, v, B, Hq, Hkv, 1, Skv,
                                   d, sc, False)
    compare(o, ref.reshape(B, Hq, d), f"decode gqa {shape}")
    if Hq // Hkv < 4:
        # the VALU kernel sums unrounded fp32 probabilities: fp32-accurate lse
        compare(lse, ref_lse.reshape(B, Hq), f"decode gqa lse {shape}", max_abs=1e-4,
                mean_abs=2e-5)
    else:
        # the matrix-core kernel sums the bf16-rounded probabilities (as prefill)
        compare(lse, ref_lse.reshape(B, Hq), f"decode gqa lse {shape}", max_abs=LSE_MAX_ABS,
                mean_abs=LSE_MEAN_ABS)


@pytest.mark.parametrize("d", [64, 128])
def test_decode_gqa_closed_forms(pa, d):
    # matrix-core decode: identical V rows give that row exactly (the weights
    # are an exact convex combination); Q = 0 gives the column mean of V and
    # lse = log(Skv)
    B, Hq, Hkv, Skv = 2, 16, 2, 777
    q = random_bf16((B, Hq, d), 1600)
    k = random_bf16((B, Hkv, Skv, d), 1601)
    row = random_bf16((B, Hkv, 1, d), 1602)
    v_same = row.expand(B, Hkv, Skv, d).contiguous()
    announce(f"attn_decode_ex gqa closed forms d={d}")
    o = pa.attn_decode(q.to(DEV), k.to(DEV), v_same.to(DEV))
    v = random_bf16((B, Hkv, Skv, d), 1603)
    o0, lse0 = pa.attn_decode(torch.zeros_like(q).to(DEV), k.to(DEV), v.to(DEV), return_lse=True)
    torch.cuda.synchronize()
    want = row.float().repeat_interleave(Hq // Hkv, dim=1).reshape(B, Hq, d)
    np.testing.assert_allclose(o.cpu().double().numpy(), want.double().numpy(), atol=2e-6,
                               rtol=1e-6)
    mean = v.double().mean(dim=2).repeat_interleave(Hq // Hkv, dim=1)
    compare(o0, mean.numpy(), "Q = 0 gives the mean of V", max_abs=2e-3, mean_abs=2e-4)
    np.testing.assert_allclose(lse0.cpu().double().numpy(), math.log(Skv), atol=2e-6, rtol=0)


def test_decode_gqa_split_invariance(pa):
    B, Hq, Hkv, Skv, d = 1, 16, 2, 5000, 128
    q = random_bf16((B, Hq, d), 1700).to(DEV)
    k = random_bf16((B, Hkv, Skv, d), 1701).to(DEV)
    v = random_bf16((B, Hkv, Skv, d), 1702).to(DEV)
    announce("attn_decode_ex gqa split counts")
    outs = {n: pa.attn_decode(q, k, v, n_splits=n) for n in (1, 3, 16, 40)}
    torch.cuda.synchronize()
    ref, _ = oracle.attn_gqa(q.cpu().reshape(B, Hq, 1, d).contiguous(), k.cpu(), v.cpu(), B, Hq,
                             Hkv, 1, Skv, d, float(np.float32(1.0 / math.sqrt(d))), False)
    for n, o in outs.items():
        compare(o, ref.reshape(B, Hq, d), f"splits {n} vs oracle")
        # the splits change only which reference max each probability is rounded against
        compare(o, outs[1].cpu().double().numpy(), f"splits {n} vs 1", max_abs=2e-3, mean_abs=2e-4)


def test_decode_caller_workspace(pa):
    B, Hq, Hkv, Skv, d = 2, 8, 2, 3000, 128
    q = random_bf16((B, Hq, d), 1100).to(DEV)
    k, v = random_bf16((B, Hkv, Skv, d), 1101).to(DEV), random_bf16((B, Hkv, Skv, d), 1102).to(DEV)
    for n in (0, 7):
        need = pa.decode_workspace_bytes(B, Hq, Hkv, Skv, d, n)
        announce(f"attn_decode_ex caller workspace n={n} bytes={need}")
        assert need > 0
        ws = torch.empty(need, dtype=torch.uint8, device=DEV)
        a = pa.attn_decode(q, k, v, n_splits=n)
        b = pa.attn_decode(q, k, v, n_splits=n, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(a.cpu(), b.cpu()), "caller workspace changes the result"
        small = torch.empty(need - 16, dtype=torch.uint8, device=DEV)
        with pytest.raises(pa.AttnError) as e:
            pa.attn_decode(q, k, v, n_splits=n, workspace=small)
        assert e.value.code == pa.ATTN_EINVAL


# ---------------------------------------------------------------- key splits
class forced_split_plan(forced_plan):
    def __init__(self, bn: int, waves: int, pipe: int, splits: int):
        super().__init__(bn, waves, pipe)
        self.value += f",splits={splits}"


SPLIT_VARIANTS = [(32, 4, 0, 3), (32, 8, 3, 5), (64, 4, 1, 2), (64, 8, 3, 4), (64, 8, 1, 6),
                  (128, 8, 1, 3), (128, 4, 0, 2)]


@pytest.mark.parametrize("variant", SPLIT_VARIANTS, ids=[str(v) for v in SPLIT_VARIANTS])
def test_fwd_key_splits_every_schedule(pa, variant):
    # ragged query tail, key count that leaves a short last split, grouped heads
    B, Hq, Hkv, Sq, Skv = 2, 4, 2, 77, 1000
    for d in (64, 128):
        q, k, v = _qkv(B, Hq, Hkv, Sq, Skv, d, 1200 + d)
        sc = float(np.float32(1.0 / math.sqrt(d)))
        announce(f"attn_fwd_ex key splits {variant} d={d}")
        with forced_split_plan(*variant):
            o, lse = pa.attn_fwd(q.to(DEV), k.to(DEV), v.to(DEV), scale=sc, return_lse=True)
            o16 = pa.attn_fwd(q.to(DEV), k.to(DEV), v.to(DEV), scale=sc,
                              out_dtype=torch.bfloat16)
        torch.cuda.synchronize()
        ref, ref_lse = oracle.attn_gqa(q, k, v, B, Hq, Hkv, Sq, Skv, d, sc, False)
        compare(o, ref, f"splits {variant} d={d}")
        compare(o16.float(), ref, f"splits {variant} d={d} bf16")
        assert torch.equal(o16.cpu(), o.cpu().to(torch.bfloat16))
        compare(lse, ref_lse, f"splits {variant} d={d} lse", max_abs=LSE_MAX_ABS,
                mean_abs=LSE_MEAN_ABS)


def test_fwd_key_splits_one_key_in_last_split(pa):
    # Skv = 2*64 + 1 with 3 splits of 64 keys: the last split holds one key
    B, H, Sq, Skv, d = 1, 3, 130, 129, 128
    q, k, v = _qkv(B, H, H, Sq, Skv, d, 1300)
    sc = float(np.float32(1.0 / math.sqrt(d)))
    announce("attn_fwd_ex key splits, one-key split")
    with forced_split_plan(64, 8, 1, 3):
        o = pa.attn_fwd(q.to(DEV), k.to(DEV), v.to(DEV), scale=sc)
    torch.cuda.synchronize()
    compare(o, oracle.attn(q, k, v, B, H, Sq, Skv, d, sc, False), "one-key split")


@pytest.mark.parametrize("variant", [(64, 8, 3, 256), (128, 4, 1, 96), (32, 8, 1, 192)],
                         ids=["64x8x3_256", "128x4x1_96", "32x8x1_192"])
def test_fwd_many_key_splits(pa, variant):
    # more splits than the 32 the combine saw before: one q-tile of a few
    # queries against a long key range, the last split short
    bn, waves, pipe, n = variant
    B, H, Sq, d = 1, 2, 40, 128
    Skv = n * 2 * bn - bn // 2  # chunk 2*bn, every split non-empty, the last half full
    q, k, v = _qkv(B, H, H, Sq, Skv, d, 1350 + n)
    sc = float(np.float32(1.0 / math.sqrt(d)))
    announce(f"attn_fwd_ex many key splits {variant} Skv={Skv}")
    with forced_split_plan(bn, waves, pipe, n):
        o, lse = pa.attn_fwd(q.to(DEV), k.to(DEV), v.to(DEV), scale=sc, return_lse=True)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.attn_gqa(q, k, v, B, H, H, Sq, Skv, d, sc, False)
    compare(o, ref, f"{n} splits", rel_fro=1e-2)
    compare(lse, ref_lse, f"{n} splits lse", max_abs=LSE_MAX_ABS, mean_abs=LSE_MEAN_ABS)


def test_fwd_key_splits_chosen_by_the_planner(pa):
    # few heads and queries against many keys: the planner splits the keys
    B, H, Sq, Skv, d = 1, 2, 256, 12000, 128
    plan = pa.parse_plan(pa.get_plan(pa.KIND_FWD, B, H, Sq, Skv, d, False))
    announce(f"attn_fwd planner split {plan}")
    assert plan["KV_SPLITS"] > 1, plan
    q, k, v = _qkv(B, H, H, Sq, Skv, d, 1400)
    sc = float(np.float32(1.0 / math.sqrt(d)))
    o, lse = pa.attn_fwd(q.to(DEV), k.to(DEV), v.to(DEV), scale=sc, return_lse=True)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.attn_gqa(q, k, v, B, H, H, Sq, Skv, d, sc, False)
    compare(o, ref, "planner split")
    compare(lse, ref_lse, "planner split lse", max_abs=LSE_MAX_ABS, mean_abs=LSE_MEAN_ABS)


def test_fwd_key_splits_after_decode_share_the_workspace(pa):
    # decode and split prefill on one stream reuse the per-stream workspace
    B, H, Sq, Skv, d = 1, 2, 64, 5000, 64
    q, k, v = _qkv(B, H, H, Sq, Skv, d, 1500)
    qd = random_bf16((B, H, d), 1501)
    sc = float(np.float32(1.0 / math.sqrt(d)))
    announce("split prefill interleaved with decode")
    kd, vd = k.to(DEV), v.to(DEV)
    with forced_split_plan(64, 4, 1, 6):
        outs = []
        for _ in range(3):
            outs.append(pa.attn_fwd(q.to(DEV), kd, vd, scale=sc))
            dec = pa.attn_decode(qd.to(DEV), kd, vd)
    torch.cuda.synchronize()
    for o in outs[1:]:
        assert torch.equal(o.cpu(), outs[0].cpu())
    compare(outs[0], oracle.attn(q, k, v, B, H, Sq, Skv, d, sc, False), "split prefill")
    ref_d = oracle.attn(qd.reshape(B, H, 1, d).contiguous(), k, v, B, H, 1, Skv, d, sc, False)
    compare(dec, ref_d.reshape(B, H, d), "decode between")


def test_two_streams_keep_separate_workspaces(pa):
    # decode on one stream and split-key prefill on another, issued alternately
    # so that both are in flight together: each stream's partials live in its
    # own workspace, so neither result is disturbed by the other
    B, H, Sq, Skv, d = 2, 4, 96, 3000, 128
    q, k, v = _qkv(B, H, H, Sq, Skv, d, 1600)
    qd = random_bf16((B, H, d), 1603)
    sc = float(np.float32(1.0 / math.sqrt(d)))
    qg, kg, vg, qdg = q.to(DEV), k.to(DEV), v.to(DEV), qd.to(DEV)
    torch.cuda.synchronize()
    s_dec, s_fwd = torch.cuda.Stream(), torch.cuda.Stream()
    announce("decode and split prefill on two streams")
    decs, fwds = [], []
    with forced_split_plan(64, 4, 1, 8):
        for _ in range(4):
            with torch.cuda.stream(s_dec):
                decs.append(pa.attn_decode(qdg, kg, vg, n_splits=12))
            with torch.cuda.stream(s_fwd):
                fwds.append(pa.attn_fwd(qg, kg, vg, scale=sc))
    torch.cuda.synchronize()
    for o in decs[1:]:
        assert torch.equal(o.cpu(), decs[0].cpu())
    for o in fwds[1:]:
        assert torch.equal(o.cpu(), fwds[0].cpu())
    compare(fwds[0], oracle.attn(q, k, v, B, H, Sq, Skv, d, sc, False), "split prefill stream")
    ref_d = oracle.attn(qd.reshape(B, H, 1, d).contiguous(), k, v, B, H, 1, Skv, d, sc, False)
    compare(decs[0], ref_d.reshape(B, H, d), "decode stream")


def test_fwd_key_splits_rejected_for_causal(pa):
    q = torch.zeros((1, 1, 64, 64), dtype=torch.bfloat16, device=DEV)
    with forced_split_plan(64, 8, 1, 2):
        with pytest.raises(pa.AttnError) as e:
            pa.attn_fwd(q, q, q, causal=True)
    assert e.value.code == pa.ATTN_EINVAL


# ---------------------------------------------------------------- causal chunks
class forced_chunk_plan(forced_plan):
    def __init__(self, bn: int, waves: int, pipe: int, splits: int, fold: int,
                 form: int = 0):
        super().__init__(bn, waves, pipe)
        self.value += f",splits={splits},fold={fold},form={form}"


# B, Hq, Hkv, Sq, Skv, splits, folded heads: one query; a group whose rows end
# inside a 32-row wave and wrap within one; a chunk of exactly one q-tile;
# several q-tiles with a ragged end; the diagonal at the very start of the last
# split; more splits than tiles a wave is active in
CHUNKS = [(1, 4, 1, 1, 2, 1, 4), (2, 6, 2, 11, 130, 1, 3), (1, 4, 1, 33, 260, 2, 4),
          (2, 2, 2, 256, 512, 2, 1), (1, 2, 1, 300, 700, 2, 1), (1, 8, 2, 70, 500, 3, 4),
          (1, 1, 1, 64, 128, 2, 1), (1, 5, 5, 17, 1100, 6, 1)]


@pytest.mark.parametrize("tile", [(64, 8, 3), (64, 4, 1), (32, 4, 1)])
@pytest.mark.parametrize("d", [64, 128])
def test_fwd_causal_chunk(pa, tile, d):
    for i, (B, Hq, Hkv, Sq, Skv, splits, fold) in enumerate(CHUNKS):
        q, k, v = _qkv(B, Hq, Hkv, Sq, Skv, d, 1500 + 7 * i + d)
        qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
        sc = float(np.float32(1.0 / math.sqrt(d)))
        announce(f"attn_fwd_ex causal chunk {tile} d={d} {CHUNKS[i]}")
        with forced_chunk_plan(*tile, splits, fold):
            o, lse = pa.attn_fwd(qd, kd, vd, causal=True, return_lse=True)
            o16 = pa.attn_fwd(qd, kd, vd, causal=True, out_dtype=torch.bfloat16)
        torch.cuda.synchronize()
        ref, ref_lse = oracle.attn_gqa(q, k, v, B, Hq, Hkv, Sq, Skv, d, sc, True)
        compare(o, ref, f"chunk {tile} d={d} {CHUNKS[i]}")
        compare(lse, ref_lse, f"chunk {tile} d={d} {CHUNKS[i]} lse", max_abs=LSE_MAX_ABS,
                mean_abs=LSE_MEAN_ABS)
        assert torch.equal(o16.cpu(), o.cpu().to(torch.bfloat16))


# B, Hq, Hkv, Sq, Skv: heads that the XCDs share evenly (8, 16) or not; one
# q-tile, its edge and one row past it; a short cache before the chunk
SINGLES = [(1, 1, 1, 1, 1), (1, 3, 1, 256, 256), (2, 4, 2, 257, 257), (2, 8, 2, 300, 333),
           (1, 5, 5, 700, 800), (1, 8, 8, 513, 513)]


@pytest.mark.parametrize("tile", [(64, 8, 3), (64, 4, 1), (32, 4, 1)])
@pytest.mark.parametrize("d", [64, 128])
def test_fwd_causal_single_tiles(pa, tile, d):
    for i, (B, Hq, Hkv, Sq, Skv) in enumerate(SINGLES):
        q, k, v = _qkv(B, Hq, Hkv, Sq, Skv, d, 1900 + 7 * i + d)
        qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
        sc = float(np.float32(1.0 / math.sqrt(d)))
        announce(f"attn_fwd_ex causal single q-tiles {tile} d={d} {SINGLES[i]}")
        with forced_chunk_plan(*tile, 1, 1, form=1):
            o, lse = pa.attn_fwd(qd, kd, vd, causal=True, return_lse=True)
        torch.cuda.synchronize()
        ref, ref_lse = oracle.attn_gqa(q, k, v, B, Hq, Hkv, Sq, Skv, d, sc, True)
        compare(o, ref, f"singles {tile} d={d} {SINGLES[i]}")
        compare(lse, ref_lse, f"singles {tile} d={d} {SINGLES[i]} lse", max_abs=LSE_MAX_ABS,
                mean_abs=LSE_MEAN_ABS)


# B, Hq, Hkv, Sq, Skv, splits, by the rows of a q-tile: a split per q-tile and one more
# row; splits that end inside, at and past a q-tile's first row; a cache shorter than the
# chunk; early q-tiles of one split and late ones of all; grouped heads; chains that the
# combine walks in parallel (8 and 16 splits, up to 2048 rows and more)
TRIANGLES = {256: [(1, 1, 1, 513, 513, 2), (2, 4, 2, 1100, 1100, 4), (1, 3, 1, 2048, 2048, 8),
                   (1, 2, 2, 700, 900, 3), (1, 1, 1, 4096, 4096, 16), (1, 2, 1, 1400, 1790, 6)],
             128: [(1, 1, 1, 257, 257, 2), (2, 4, 2, 650, 650, 4), (1, 3, 1, 1024, 1024, 8),
                   (1, 2, 2, 400, 520, 3), (1, 1, 1, 2048, 2048, 16), (1, 2, 1, 700, 760, 6)]}


@pytest.mark.parametrize("tile", [(64, 8, 3), (64, 4, 1), (32, 4, 1)])
@pytest.mark.parametrize("d", [64, 128])
def test_fwd_causal_split_triangle(pa, tile, d):
    for i, (B, Hq, Hkv, Sq, Skv, splits) in enumerate(TRIANGLES[32 * tile[1]]):
        q, k, v = _qkv(B, Hq, Hkv, Sq, Skv, d, 2100 + 7 * i + d)
        qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
        sc = float(np.float32(1.0 / math.sqrt(d)))
        what = (B, Hq, Hkv, Sq, Skv, splits)
        announce(f"attn_fwd_ex causal split triangle {tile} d={d} {what}")
        # NaN in every partial of the workspace, laid out alike (the same rows and
        # splits): where no split of a row writes, none may be read
        with forced_split_plan(*tile, splits):
            poison = pa.attn_fwd(torch.full_like(qd, float("nan")), kd, vd)
        with forced_chunk_plan(*tile, splits, 1, form=2):  # (refused if it were infeasible)
            o, lse = pa.attn_fwd(qd, kd, vd, causal=True, return_lse=True)
            o16 = pa.attn_fwd(qd, kd, vd, causal=True, out_dtype=torch.bfloat16)
        torch.cuda.synchronize()
        assert torch.isnan(poison).all()
        ref, ref_lse = oracle.attn_gqa(q, k, v, B, Hq, Hkv, Sq, Skv, d, sc, True)
        compare(o, ref, f"triangle {tile} d={d} {what}")
        compare(lse, ref_lse, f"triangle {tile} d={d} {what} lse", max_abs=LSE_MAX_ABS,
                mean_abs=LSE_MEAN_ABS)
        assert torch.equal(o16.cpu(), o.cpu().to(torch.bfloat16))


@pytest.mark.parametrize("causal", [False, True])
def test_fwd_folded_heads_by_plan(pa, causal):
    # the planner's own choice where folding the group fills the q-tile
    B, Hq, Hkv, Sq, Skv, d = 2, 16, 2, 9, 3000, 128
    q, k, v = _qkv(B, Hq, Hkv, Sq, Skv, d, 1700)
    assert call_plan(pa, B, Hq, Hkv, Sq, Skv, d, causal)["FOLD"] == Hq // Hkv
    announce(f"attn_fwd_ex folded heads causal={causal}")
    o, lse = pa.attn_fwd(q.to(DEV), k.to(DEV), v.to(DEV), scale=-0.1, causal=causal,
                         return_lse=True)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.attn_gqa(q, k, v, B, Hq, Hkv, Sq, Skv, d, float(np.float32(-0.1)),
                                   causal)
    compare(o, ref, f"folded causal={causal}")
    compare(lse, ref_lse, f"folded causal={causal} lse", max_abs=LSE_MAX_ABS,
            mean_abs=LSE_MEAN_ABS)


def test_fwd_causal_chunk_in_a_graph(pa):
    # replays stay right after an eager call of the same stream has grown the
    # workspace (that the captured call uses none is checked on its plan, in
    # test_fwd_in_a_graph_uses_no_workspace)
    B, Hq, Hkv, Sq, Skv, d = 1, 4, 1, 64, 4096, 128
    q, k, v = _qkv(B, Hq, Hkv, Sq, Skv, d, 1800)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    o = torch.empty((B, Hq, Sq, d), dtype=torch.float32, device=DEV)
    ref = oracle.attn_gqa(q, k, v, B, Hq, Hkv, Sq, Skv, d, float(np.float32(1 / math.sqrt(d))),
                          True)[0]
    announce("attn_fwd causal chunk captured")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        pa.attn_fwd(qd, kd, vd, o=o, causal=True)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        pa.attn_fwd(qd, kd, vd, o=o, causal=True)
    for rows in (64, 512, 1024):
        o.fill_(float("nan"))
        with torch.cuda.stream(side):
            big = torch.zeros((1, 32, rows, d), dtype=torch.bfloat16, device=DEV)
            kv = torch.zeros((1, 32, 4 * rows, d), dtype=torch.bfloat16, device=DEV)
            pa.attn_fwd(big, kv, kv, causal=True)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        compare(o, ref, f"replay after an eager call of {rows} rows")


def call_plan(pa, B, Hq, Hkv, Sq, Skv, d, causal):
    """The plan that a call on the current stream would run now."""
    buf = ctypes.create_string_buffer(512)
    pa.lib.attn_set_stream(torch.cuda.current_stream().cuda_stream)
    rc = pa.lib.attn__fwd_call_plan(B, Hq, Hkv, Sq, Skv, d, int(causal), buf, 512)
    assert rc > 0, pa.last_error()
    return pa.parse_plan(buf.value.decode())


# B, Hq, Hkv, Sq, Skv, causal: each splits its keys in an eager call -- few heads,
# folded heads of a short chunk, a longer chunk, the causal triangle
GRAPH_SHAPES = [(1, 2, 2, 700, 4096, False), (1, 8, 1, 16, 8000, False),
                (1, 4, 1, 64, 4096, True), (1, 2, 2, 2048, 2048, True)]


@pytest.mark.parametrize("shape", GRAPH_SHAPES, ids=lambda s: "x".join(map(str, s[:5])))
def test_fwd_in_a_graph_uses_no_workspace(pa, shape):
    # the invariant is checked on the plan: a replay that used a released workspace
    # could still give the right result
    B, Hq, Hkv, Sq, Skv, causal = shape
    d = 128
    q, k, v = _qkv(B, Hq, Hkv, Sq, Skv, d, 2300 + Sq)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    o = torch.empty((B, Hq, Sq, d), dtype=torch.float32, device=DEV)
    ref = oracle.attn_gqa(q, k, v, B, Hq, Hkv, Sq, Skv, d, float(np.float32(1 / math.sqrt(d))),
                          causal)[0]
    args = (B, Hq, Hkv, Sq, Skv, d, causal)
    announce(f"attn_fwd {args} captured")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert call_plan(pa, *args)["KV_SPLITS"] > 1
        pa.attn_fwd(qd, kd, vd, o=o, causal=causal)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        assert call_plan(pa, *args)["KV_SPLITS"] == 1
        pa.attn_fwd(qd, kd, vd, o=o, causal=causal)
    for heads in (2, 4):
        o.fill_(float("nan"))
        with torch.cuda.stream(side):  # grows the stream's workspace
            big = torch.zeros((1, heads, 4096, d), dtype=torch.bfloat16, device=DEV)
            pa.attn_fwd(big, big, big)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        compare(o, ref, f"replay {args} after an eager call of {heads} heads")


@pytest.mark.parametrize("shape", GRAPH_SHAPES + [(2, 16, 2, 9, 3000, True), (4, 16, 16, 512, 512, True)],
                         ids=lambda s: "x".join(map(str, s[:5])))
def test_plan_query_reports_the_plan_that_runs(pa, shape):
    B, Hq, Hkv, Sq, Skv, causal = shape
    assert call_plan(pa, B, Hq, Hkv, Sq, Skv, 128, causal) == pa.parse_plan(
        pa.get_plan(pa.KIND_FWD, B, Hq, Sq, Skv, 128, causal, Hkv=Hkv))


# key splits and rows on both sides of where the combine gives each row a workgroup: 8
# splits up to 2048 rows, past them chains of 2048 / d splits
@pytest.mark.parametrize("d,rows,splits", [(128, 2047, 6), (128, 2048, 8), (128, 2049, 8),
                                           (128, 2049, 12), (128, 2049, 16), (64, 2048, 8),
                                           (64, 2049, 24), (64, 2049, 32)])
def test_fwd_split_combine_forms(pa, d, rows, splits):
    B, H, Skv = 1, 1, 32 * splits - 5
    q, k, v = _qkv(B, H, H, rows, Skv, d, 2600 + splits)
    sc = float(np.float32(1.0 / math.sqrt(d)))
    announce(f"split combine d={d} rows={rows} splits={splits}")
    with forced_split_plan(32, 4, 1, splits):
        o, lse = pa.attn_fwd(q.to(DEV), k.to(DEV), v.to(DEV), return_lse=True)
        o16 = pa.attn_fwd(q.to(DEV), k.to(DEV), v.to(DEV), out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.attn_gqa(q, k, v, B, H, H, rows, Skv, d, sc, False)
    compare(o, ref, f"combine d={d} rows={rows} splits={splits}")
    compare(lse, ref_lse, f"combine lse d={d} rows={rows} splits={splits}", max_abs=LSE_MAX_ABS,
            mean_abs=LSE_MEAN_ABS)
    assert torch.equal(o16.cpu(), o.cpu().to(torch.bfloat16))
