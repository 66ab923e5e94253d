"""The attention forward on its own stashed operands: ctx and the log-sum-exp of
a layer call against float64 attention over the stashed Q, K, V, with scores of
ordinary size and of a size where a row's maximum grows by many powers of two
from tile to tile,
at sequence lengths around the 64-key and 128-query tiles and both head sizes.

Bound: the products are exact in fp32 and P carries about 16 bits (2^-16 of
sum P |V|, at most max |V|), so ctx is within one bf16 step (2^-8) of its value
plus 2^-15 max |V|; the log-sum-exp, whose scores are fp32 sums, within 2^-18
of the largest score plus 1e-5."""
import math

import pytest
import torch

import workloads as W
from gpu_common import Buffers
import paper_2411_06465_amd as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 12.0])
@pytest.mark.parametrize("d,seq,cp", [(64, 64, 1), (64, 193, 1), (128, 129, 1), (128, 520, 1), (128, 512, 2)])
def test_forward_matches_float64_attention(d, seq, cp, scale):
    print(f"\n[attention scores d={d} s={seq} cp={cp} scale={scale}]", flush=True)
    w = W.LayerWorkload(f"scores-{d}-{seq}-{cp}", 4 * d, 4, 2, 256, seq, cp=cp, cp_rank=cp - 1, n_gpus=cp)
    buf = Buffers(w)
    buf.weights["qkv"].mul_(scale)
    st = L.llama_layer_fwd(buf.model, buf.par, buf.weights, buf.x, buf.y, buf.arena, peers=buf.peers)
    q, k, v, ctx = (buf.stash_view(st, n, (1, w.s_c, -1)).clone() for n in ("q", "k", "v", "ctx"))
    lse = buf.stash_view(st, "lse", (1, 4, w.s_c), torch.float32).clone()
    torch.cuda.synchronize()
    st.release()
    pos = torch.arange(seq).cuda()
    rest = pos[:0]
    if cp > 1:
        n, own = seq // (2 * cp), (w.cp_rank, 2 * cp - 1 - w.cp_rank)
        chunks = pos.view(2 * cp, n)
        pos = torch.cat([chunks[i] for i in own])
        rest = torch.cat([chunks[i] for i in range(2 * cp) if i not in own])
        k = torch.cat([k, buf.peers["remote_k"].view(1, -1, k.shape[-1])], 1)
        v = torch.cat([v, buf.peers["remote_v"].view(1, -1, v.shape[-1])], 1)
    mask = torch.cat([pos, rest])[None] > pos[:, None]
    for h in range(4):
        qh, c = q[0, :, h * d:(h + 1) * d].double(), ctx[0, :, h * d:(h + 1) * d].double()
        kh, vh = (t[0, :, h // 2 * d:(h // 2 + 1) * d].double() for t in (k, v))
        s = (qh @ kh.T / math.sqrt(d)).masked_fill(mask, -math.inf)
        ref = s.softmax(-1) @ vh
        bound = 2.0 ** -8 * ref.abs() + 2.0 ** -15 * vh.abs().max()
        assert bool(((c - ref).abs() <= bound).all()), (h, float(((c - ref).abs() / bound).max()))
        big = float(s.masked_fill(mask, 0).abs().max())
        assert float((lse[0, h].double() - s.logsumexp(-1)).abs().max()) <= 2.0 ** -18 * big + 1e-5


@pytest.mark.parametrize("d", [64, 128])
def test_log_sum_exp_of_a_row_whose_maximum_comes_late(d):
    """Key 0 has a score near -5, key 64, the first of the second tile, one near
    0.3, and the others none to speak of: the row sum is 1 + 2^-7 or so, and the
    log-sum-exp that score plus 2^-7.  With the exact maximum as the reference the
    only rounding of its size is that of the sum: half a step of [1, 2), at most
    2^-24, and the rms over the rows below that.  A reference left at the first
    tile's maximum, 2^7 too low, puts the rounding of an exponent near 7 and of
    the logarithm of a sum near 128 into it instead, 2^-22 each."""
    print(f"\n[attention late maximum d={d}]", flush=True)
    w = W.LayerWorkload(f"late-{d}", 4 * d, 4, 2, 256, 128, rope_base=1e12)
    buf = Buffers(w)
    # only the slowest RoPE pair of a head is used: a score is the product of two features of equally long rows
    qkv, x, j = buf.weights["qkv"], buf.x, d // 2 - 1
    qkv[:6 * d].zero_()
    qkv[j:4 * d:d, 1] = torch.tensor([9.0, 9.25, 9.5, 9.75], device="cuda").mul(math.sqrt(d / 64)).to(torch.bfloat16)
    qkv[4 * d + j:6 * d:d, 0] = 1.0
    buf.weights["norm1"].fill_(1.0)
    key = torch.full((128,), -20.0, device="cuda")
    key[0], key[64] = -2.0, 0.12
    rest = torch.randn(128, 4 * d - 2, generator=torch.Generator("cuda").manual_seed(d), device="cuda")
    rest *= ((2 * 4 * d - 16 - key.square()).sqrt() / rest.norm(dim=1))[:, None]
    x[0] = torch.cat([key[:, None], torch.full((128, 1), 4.0, device="cuda"), rest], 1).to(torch.bfloat16)
    st = L.llama_layer_fwd(buf.model, buf.par, buf.weights, x, buf.y, buf.arena)
    q, k = (buf.stash_view(st, n, (128, -1, d)).double() for n in ("q", "k"))
    lse = buf.stash_view(st, "lse", (4, 128), torch.float32).double()
    torch.cuda.synchronize()
    st.release()
    for h in range(4):
        s = ((q[64:, h].cpu() @ k[:, h // 2].cpu().T) / math.sqrt(d)).masked_fill_(
            torch.ones(64, 128, dtype=torch.bool).triu(65), -math.inf)
        gap = (s[:, 64] - s[:, 0]) / math.log(2.0)
        assert 6.0 < float(gap.min()) and float(gap.max()) < 7.9, (float(gap.min()), float(gap.max()))
        err = lse[h, 64:].cpu() - s.logsumexp(-1)
        print(f"head {h}: gap 2^{float(gap.mean()):.2f}, rms {float(err.square().mean().sqrt()):.2e}", flush=True)
        assert float(err.square().mean().sqrt()) <= 2.0 ** -24
