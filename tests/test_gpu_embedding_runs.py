"""GPU parity of the embedding gradient where its sorted runs can go wrong:
token counts around a sort chunk (2048) and the unsorted limits (512 tokens, 2^20
elements in the rank's share of the rows), hidden sizes that are no multiple of a
column block (1024), one id on every token, no id in range, against a float64
sum.  fp32 sums of at most n terms of either
sign: within n * 2^-24 of the sum of magnitudes."""
import numpy as np
import pytest
import torch

import paper_2411_06465_amd as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,ids", [(8, 256, "mixed"), (512, 256, "mixed"), (520, 1280, "mixed"), (2048, 256, "same"),
                                     (2056, 256, "mixed"), (4104, 768, "same"), (2056, 256, "none"),
                                     # enough elements for the sort: whole chunks, one past a chunk, three chunks
                                     (2048, 2304, "same"), (2056, 2304, "mixed"), (4104, 1280, "mixed"),
                                     (2056, 2304, "none")])
def test_gradient_matches_float64(n, h, ids):
    print(f"\n[embedding runs n={n} h={h} {ids}]", flush=True)
    v, t, rank = 4000, 4, 1
    v_t = v // t
    rng = np.random.default_rng(n + h)
    if ids == "same":
        tok = np.full(n, rank * v_t + 7)
    elif ids == "none":
        tok = rng.integers(0, v_t, n)
    else:
        tok = np.where(rng.random(n) < 0.3, rank * v_t + v_t - 1, rng.integers(0, v, n))
    model, par = L.make_model(h, h // 64, h // 64, 32, vocab=v), L.make_parallel(n, tp=t, tp_rank=rank)
    own, peer = n // t, n - n // t
    dx = torch.randn(1, own, h, device="cuda").to(torch.bfloat16)
    pdx = torch.randn(1, peer, h, device="cuda").to(torch.bfloat16)
    table = torch.randn(v_t, h, device="cuda").to(torch.bfloat16)
    buf = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    arena = L.Arena.on(buf)
    ids_t = torch.from_numpy(tok.astype(np.int64)).cuda().view(1, n)
    x = torch.empty(1, own, h, dtype=torch.bfloat16, device="cuda")
    send = torch.empty(1, peer, h, dtype=torch.bfloat16, device="cuda")
    st = L.embedding_fwd(model, par, ids_t, table, x, arena, send=send)
    dw = torch.ones(v_t, h, device="cuda")
    L.embedding_bwd(model, par, st, dx, dw, arena, peer_dx=pdx)
    torch.cuda.synchronize()
    assert arena.stats()["in_use"] == 0
    assert torch.equal(ids_t.cpu().view(-1), torch.from_numpy(tok.astype(np.int64)))   # the caller's ids stay
    full = torch.cat([pdx[:, :rank * own], dx, pdx[:, rank * own:]], 1)[0].double()
    local = ids_t.view(-1) - rank * v_t
    hit = (local >= 0) & (local < v_t)
    ref = torch.ones(v_t, h, device="cuda", dtype=torch.float64).index_add_(0, local[hit], full[hit])
    mag = torch.ones(v_t, h, device="cuda", dtype=torch.float64).index_add_(0, local[hit], full[hit].abs())
    assert bool(((dw.double() - ref).abs() <= n * 2.0 ** -24 * mag).all())


def test_captured_backward_replays_on_kept_ids_and_full_arena_runs():
    """A captured backward adds the same gradient on every replay (the stashed
    ids stay as they are), and an arena that holds the ids alone still runs the
    call, in token order.  Small whole numbers: every sum is exact in fp32."""
    n, h, v = 4104, 256, 1000
    rng = np.random.default_rng(3)
    tok = torch.from_numpy(np.where(rng.random(n) < 0.3, 7, rng.integers(0, v, n)).astype(np.int64)).cuda()
    model, par = L.make_model(h, h // 64, h // 64, 32, vocab=v), L.make_parallel(n)
    dx = torch.randint(-4, 5, (1, n, h), device="cuda").to(torch.bfloat16)
    table, x = torch.zeros(v, h, dtype=torch.bfloat16, device="cuda"), torch.empty(1, n, h, dtype=torch.bfloat16,
                                                                                  device="cuda")
    once = torch.zeros(v, h, device="cuda").index_add_(0, tok, dx[0].float())
    for nbytes in (1 << 20, (8 * n + 255) // 256 * 256):
        arena = L.Arena.on(torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
        dw = torch.zeros(v, h, device="cuda")
        st = L.embedding_fwd(model, par, tok.view(1, n), table, x, arena)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            L.embedding_bwd(model, par, st, dx, dw, arena, stream=torch.cuda.current_stream())
        assert arena.stats()["in_use"] == 0
        for i in range(1, 4):
            graph.replay()
            torch.cuda.synchronize()
            print(f"\n[embedding replay arena={nbytes} {i}]", flush=True)
            assert torch.equal(dw, i * once)


@pytest.mark.parametrize("n,h,t,sorts", [(512, 8192, 1, False), (1024, 512, 1, False), (4096, 512, 4, False),
                                         (4096, 256, 1, True), (1024, 4096, 4, True), (520, 8192, 4, True)])
def test_only_calls_with_enough_rows_sort(n, h, t, sorts):
    """A call that adds fewer than 2^20 elements takes no workspace: its sort would take longer than its adds."""
    print(f"\n[embedding sort rule n={n} h={h} tp={t}]", flush=True)
    v = 1024
    model, par = L.make_model(h, h // 64, h // 64, 32, vocab=v), L.make_parallel(n, tp=t)
    arena = L.Arena.on(torch.empty(1 << 20, dtype=torch.uint8, device="cuda"))
    ids = torch.arange(n, device="cuda").remainder_(v).view(1, n)
    own, peer = (torch.ones(1, m, h, dtype=torch.bfloat16, device="cuda") for m in (n // t, n - n // t))
    x, send = torch.empty_like(own), torch.empty_like(peer) if t > 1 else None
    st = L.embedding_fwd(model, par, ids, torch.zeros(v // t, h, dtype=torch.bfloat16, device="cuda"), x, arena, send=send)
    held = arena.stats()["peak"]
    dw = torch.zeros(v // t, h, device="cuda")
    L.embedding_bwd(model, par, st, own, dw, arena, peer_dx=peer if t > 1 else None)
    torch.cuda.synchronize()
    assert arena.stats()["peak"] - held == (8 * n + 255) // 256 * 256 * sorts
    assert torch.equal(dw, torch.bincount(ids[0], minlength=v)[:v // t].float()[:, None].expand_as(dw))
