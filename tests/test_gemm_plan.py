"""The tile size and the split that gemm_plan picks, against times measured on
an MI355X (us, with the pass that adds the parts): the form picked takes at most
5% more than the fastest one measured for that product."""
import os

import pytest

import paper_2411_06465_amd as L
from gemm_plans import ACC_F32, STORE_BF16, layer_max_splits, layer_plans, plan
from workloads import LLAMA3_70B_TP8, LLAMA3_8B_TP2CP2

pytestmark = pytest.mark.skipif(not os.path.exists(L.LIB_PATH), reason="libl4d.so not built")

MEASURED = [
    # output projection dX: 70B at TP8 with 8192 tokens and TP2 with 2048, 8B at TP4 with 4096
    (8192, 1024, 8192, STORE_BF16, {(256, 2): 142, (128, 1): 150}),
    (2048, 4096, 8192, STORE_BF16, {(256, 2): 138, (128, 1): 150}),
    (4096, 2048, 4096, STORE_BF16, {(256, 2): 87, (128, 1): 77}),
    # weight gradients of gathered rows
    (8192, 1024, 8192, ACC_F32, {(256, 1): 218, (256, 2): 157, (128, 1): 160}),
    (4096, 2048, 8192, ACC_F32, {(256, 1): 222, (256, 2): 158, (128, 1): 160}),
    (768, 4096, 8192, ACC_F32, {(256, 1): 184, (256, 4): 85, (128, 1): 94}),
    (1536, 4096, 8192, ACC_F32, {(256, 1): 193, (256, 2): 131, (128, 1): 149}),
    (4096, 1024, 8192, ACC_F32, {(256, 1): 200, (256, 4): 98, (128, 1): 101}),
    (1376, 512, 8192, ACC_F32, {(256, 4): 78, (128, 4): 38, (64, 1): 47}),
    (512, 688, 16384, ACC_F32, {(256, 4): 148, (64, 2): 53, (64, 4): 45}),
    # of plain rows
    (1024, 1024, 16384, ACC_F32, {(256, 4): 103, (128, 4): 59, (64, 1): 87}),
    (512, 512, 4096, ACC_F32, {(256, 4): 38, (64, 1): 21, (64, 4): 18}),
    (2048, 5464, 1024, ACC_F32, {(256, 1): 67, (128, 1): 54}),
    (4096, 2752, 1024, ACC_F32, {(256, 1): 82, (128, 1): 52}),
]


@pytest.mark.parametrize("M,N,K,kind,times", MEASURED, ids=lambda v: str(v) if isinstance(v, int) else "")
def test_plan_is_within_five_percent_of_the_fastest_form(M, N, K, kind, times):
    form = plan(M, N, K, kind, layer_max_splits(M, N, K, kind))
    assert form in times, form
    assert times[form] <= 1.05 * min(times.values()), (form, times)


def test_the_large_shards_split_where_tests_rely_on_it():
    # the full-size parity tests are the ones that run 256-row splits of a dX and of a plain output projection
    p = layer_plans(LLAMA3_70B_TP8)
    assert p["o_dx"] == (256, 2) and p["o_dw"] == (256, 2), p
    assert layer_plans(LLAMA3_8B_TP2CP2)["o_dx"] == (128, 1)
