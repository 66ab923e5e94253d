"""GPU parity of the cross-entropy where the row length changes the kernel:
vocabulary shards around the lengths whose rows are held in registers (8192,
32768 and 65536 columns) and past them, rows whose target lies in the last
vector or on another shard.  Hidden states are unit vectors, so a logit is an
element of the head weight, exactly, and d_w holds each token's dlogits."""
import pytest
import torch

import paper_2411_06465_amd as L

pytestmark = pytest.mark.gpu

H = 256
ROWS = [8, 1000, 8192, 8200, 32768, 32776, 65536, 65544]


def problem(v_t, n):
    g = torch.Generator().manual_seed(v_t)
    wl = (4 * torch.randn(v_t, H, generator=g)).to(torch.bfloat16)
    tgt = torch.randint(0, v_t, (n,), generator=g) + v_t      # the shard starts at v_t
    tgt[0], tgt[1], tgt[2] = 2 * v_t - 1, 0, v_t
    pl, pz = torch.randn(n, generator=g), torch.randn(n, generator=g)
    z = wl[:, :n].double().T                                   # [n][v_t]
    lse = torch.logaddexp(torch.logsumexp(z, 1), pl.double())
    own = (tgt >= v_t) & (tgt < 2 * v_t)
    col = (tgt - v_t).clamp(0, v_t - 1)
    loss = lse - torch.where(own, z.gather(1, col[:, None])[:, 0], pz.double())
    p = torch.exp(z - lse[:, None])
    onehot = torch.zeros_like(p).scatter_(1, col[:, None], own.double()[:, None])
    return wl, tgt, pl, pz, loss, p, onehot


@pytest.mark.parametrize("v_t", ROWS)
def test_bf16_rows(v_t):
    print(f"\n[xent rows v_t={v_t}]", flush=True)
    n, h = 16, H
    wl, tgt, pl, pz, loss, p, onehot = problem(v_t, n)
    hid = torch.eye(n, h).to(torch.bfloat16).cuda()
    lo, dh = torch.empty(n, device="cuda"), torch.empty_like(hid)
    dw = torch.zeros(v_t, h, device="cuda")
    buf = torch.empty(L.l4d_lm_head_workspace_bytes(n, h, v_t) + (1 << 20), dtype=torch.uint8, device="cuda")
    L.lm_head_xent(hid, wl.cuda(), tgt.cuda(), lo, dh, dw, L.Arena.on(buf), vocab_start=v_t, peer_lse=pl.cuda(),
                   peer_target_logit=pz.cuda(), grad_scale=0.5)
    # a loss below 64 from fp32 sums of positive terms: 2^-20 of 64; the softmax: 2^-16 (arguments below 64 in fp32,
    # 2^-18, and the exponential's few ulps); dlogits round it, less one at the target, to bf16
    assert (lo.cpu().double() - loss).abs().max() < 64 * 2.0 ** -20
    d = dw[:, :n].cpu().double().T
    assert ((d - 0.5 * (p - onehot)).abs() <= 2.0 ** -8 * (0.5 * (p - onehot)).abs() + 2.0 ** -16 * p).all()
    assert torch.count_nonzero(dw[:, n:]) == 0


@pytest.mark.parametrize("v_t", ROWS)
def test_fp32_rows(v_t):
    print(f"\n[softmax rows v_t={v_t}]", flush=True)
    n, h = 16, H
    wl, tgt, pl, pz, loss, p, _ = problem(v_t, n)
    model = L.make_model(h, 4, 4, 32, vocab=2 * v_t)
    par = L.make_parallel(n, tp=2, tp_rank=1)
    x = torch.zeros(1, n // 2, h)
    x[0, torch.arange(n // 2), torch.arange(n // 2) + n // 2] = 256.0        # rms 16: normalised 16
    peer = torch.zeros(1, n // 2, h)
    peer[0, torch.arange(n // 2), torch.arange(n // 2)] = 1.0
    gain = torch.full((h,), 1 / 16)
    lo = torch.empty(1, n, device="cuda")
    buf = torch.empty((n * v_t * 4) + (8 << 20), dtype=torch.uint8, device="cuda")
    st = L.lm_head_fwd(model, par, x.to(torch.bfloat16).cuda(), gain.to(torch.bfloat16).cuda(), wl.cuda(),
                       tgt.view(1, n).cuda(), lo, L.Arena.on(buf), peer_xn=peer.to(torch.bfloat16).cuda(),
                       peer_lse=pl.view(1, n).cuda(), peer_target_logit=pz.view(1, n).cuda())
    torch.cuda.synchronize()
    ptr, size = st.tensor("probs")
    probs = buf[ptr - buf.data_ptr():][:size].view(torch.float32).view(n, v_t).cpu().double()
    assert (lo.cpu().double()[0] - loss).abs().max() < 64 * 2.0 ** -20
    assert ((probs - p).abs() <= 2.0 ** -16 * p).all()
