"""GPU parity of the GEMM forms at the sizes where they can go wrong, through
the layer and the LM head: tiles of 64, 128 and 256 rows with ragged edges in
M, N and K, token counts that are no multiple of 8 (the reduction length of the
weight gradients), gathered operands whose slots are and are no multiple of 64
rows, split K ranges, and float-aligned gradient accumulators.  Bar: gpu_common's."""
import pytest
import torch

import workloads as W
from oracle import lm_head as OLM
from oracle.bf16 import from_bits
from gemm_plans import layer_plans
from gpu_common import Buffers, check, compare_layer, host_f64, oracle_layer
from test_gpu_lm_head import run_lm

pytestmark = pytest.mark.gpu

LAYERS = [
    # one token past a tile, 131 % 8 = 3: 64-row tiles, the weight gradients' K ends inside an 8-group
    W.LayerWorkload("tiles-s131", 256, 4, 2, 688, 131),
    # one sequence-parallel row each of 9, gathered slots of 9 rows (many per 64-row stage), two sequences
    W.LayerWorkload("tiles-tp2-s18", 256, 4, 2, 688, 18, micro_batch=2, tp=2, tp_rank=1, n_gpus=2),
    # gathered slots of 100 rows in 64-row tiles; head size 128 in 64-column tiles
    W.LayerWorkload("tiles-tp2-s200", 512, 4, 2, 1376, 200, tp=2, tp_rank=0, n_gpus=2, rope_base=5e5),
    # 128-row tiles, one and two per CU, M = 1000 and FFN 2728 ragged; head size 64 in 128-column tiles
    W.LayerWorkload("tiles-128", 1024, 16, 4, 2728, 1000, rope_base=5e5),
    # gathered slots of one, two and three 64-row stages in 64-row tiles, two sequences
    W.LayerWorkload("tiles-tp2-s128", 256, 4, 2, 688, 128, micro_batch=2, tp=2, tp_rank=1, n_gpus=2),
    W.LayerWorkload("tiles-tp4-s512", 512, 8, 4, 1376, 512, tp=4, tp_rank=2, n_gpus=4, rope_base=5e5),
    W.LayerWorkload("tiles-tp2-s384", 512, 4, 2, 1376, 384, micro_batch=3, tp=2, tp_rank=0, n_gpus=2, rope_base=5e5),
    # gathered slots of 64 rows in 128-row tiles
    W.LayerWorkload("tiles-128-tp4", 4096, 32, 8, 2048, 256, tp=4, tp_rank=3, n_gpus=4, rope_base=5e5),
    # 256-row tiles over 200 tokens (K ragged) with gathered slots of 100 rows
    W.LayerWorkload("tiles-256-tp2", 4096, 32, 8, 6144, 200, tp=2, tp_rank=1, n_gpus=2, rope_base=5e5),
]


@pytest.mark.parametrize("w", LAYERS, ids=lambda w: w.name)
def test_layer_matches_oracle(w):
    print(f"\n[case {w.name}] tokens {w.micro_batch}x{w.s_c} s_sp {w.s_sp}", flush=True)
    buf = Buffers(w)
    saved = buf.run()
    fw, bw = oracle_layer(w, buf.wbits, buf.abits)
    ok, rep = compare_layer(w, buf, saved, fw, bw)
    assert ok, "\n".join(rep)


# Layers whose backward cuts K ranges in parts, with the products that do, as
# (rows of a tile, parts): every tile size, plain and gathered rows (slots of 512,
# parts that start inside one), and a bf16 store.  Eight short sequences, so that
# the oracle's attention stays small.
SPLITS = [
    (W.LayerWorkload("split-64-128", 256, 4, 2, 1376, 1024, micro_batch=8, rope_base=5e5),
     dict(o_dw=(64, 4), qkv_dw=(64, 4), down_dw=(64, 4), gate_up_dw=(128, 4))),
    (W.LayerWorkload("split-128-tp2", 1024, 8, 2, 64, 1024, micro_batch=8, tp=2, tp_rank=1, n_gpus=2, rope_base=5e5),
     dict(qkv_dw=(128, 4), down_dw=(64, 4))),
    (W.LayerWorkload("split-256-tp2", 2048, 16, 4, 64, 1024, micro_batch=8, tp=2, tp_rank=0, n_gpus=2, rope_base=5e5),
     dict(qkv_dw=(256, 4), o_dw=(128, 4))),
    (W.LayerWorkload("split-dx-tp4", 4096, 32, 8, 512, 128, tp=4, tp_rank=2, n_gpus=4, rope_base=5e5),
     dict(o_dx=(64, 4))),
]


@pytest.mark.parametrize("w,splits", SPLITS, ids=lambda v: getattr(v, "name", ""))
def test_layer_with_split_products_matches_oracle(w, splits):
    plans = layer_plans(w)
    assert {n: plans[n] for n in splits} == splits, plans      # else the case no longer tests what it is here for
    test_layer_matches_oracle(w)


# (tokens, hidden, vocabulary): a token count of 5 mod 8, where a row counted
# twice shows in its target's row; one row; few rows over a long vocabulary (the
# K range of d_hidden in parts), with a ragged vocabulary too
@pytest.mark.parametrize("n,h,v", [(301, 256, 1000), (1, 256, 1000), (64, 512, 16384), (72, 512, 12040)])
def test_lm_head_matches_oracle(n, h, v):
    w = W.LMHeadWorkload(f"tiles-lm-{n}-{v}", n, h, v)
    print(f"\n[case {w.name}]", flush=True)
    inp = W.lm_head_inputs(w)
    loss, dh, dw = run_lm(w, inp)
    ref = OLM.lm_head_xent(from_bits(inp["hidden"]), from_bits(inp["w_lm"]), inp["targets"], 0, None, None, 1.0 / n)
    rep, ok = [], True
    ok &= check("loss", host_f64(loss), ref["loss"], bf16=False, report=rep)
    ok &= check("d_hidden", host_f64(dh), ref["d_hidden"], report=rep)
    ok &= check("d_w_lm", host_f64(dw), ref["d_w"], bf16=False, report=rep)
    assert ok, "\n".join(rep)


def test_float_aligned_gradient_accumulators(w=W.TINY):
    # the accumulators may start at any float: the same bits as 16-byte aligned ones
    print("\n[float-aligned accumulators]", flush=True)
    buf = Buffers(w)
    buf.run(keep_stash=False)
    want = {k: v.clone() for k, v in buf.grads.items()}
    buf.grads = {k: torch.zeros(v.numel() + 1, device="cuda")[1:].view(v.shape) for k, v in want.items()}
    buf.run(keep_stash=False)
    for k, v in want.items():
        assert torch.equal(buf.grads[k], v), k


def test_float_aligned_accumulators_of_split_gradients():
    # the pass that adds the parts reads and writes the accumulator too
    w = SPLITS[0][0]
    assert min(layer_plans(w)[n][1] for n in ("o_dw", "qkv_dw", "down_dw", "gate_up_dw")) > 1
    test_float_aligned_gradient_accumulators(w)
