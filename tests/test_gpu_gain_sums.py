"""GPU parity of the norm's gain gradient where its column sums can go wrong:
fewer partial rows than waves, row counts around the 256 partial sums and
one to five blocks of columns, against a float64 sum."""
import pytest

import workloads as W
from gpu_common import check, host_f64
from test_gpu_ends import head_oracle, run_head

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seq,heads", [(8, 1), (8, 3), (40, 2), (248, 5), (256, 1), (264, 3)])
def test_gain_gradient(seq, heads):
    w = W.EndsWorkload(f"gain-{seq}-{heads}", 64 * heads, heads, heads, 64, 128, seq)
    print(f"\n[gain sums rows={w.tokens} h={w.hidden}]", flush=True)
    inp = W.ends_inputs(w)
    got = run_head(w, inp, 1.0 / w.tokens)
    _, bw = head_oracle(w, inp, 1.0 / w.tokens)
    rep = []
    assert check("d_gain", host_f64(got["d_gain"]), bw["d_gain"], bf16=False, report=rep), "\n".join(rep)
