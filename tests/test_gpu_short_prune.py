"""The single-launch forms of the mask, the mask with gather, the fixed-budget threshold and the
page assignment, at the edges of the sizes they take (and one beyond, where the general kernels
run): bit-exact against the oracle."""
import numpy as np
import pytest
import torch

from oracle import kvzap_oracle as O
from paper_2601_07891_amd import binding, synth
from tests import parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,H,T,D,w", [
    (1, 8, 127, 128, 16), (1, 8, 128, 64, 128), (1, 8, 129, 256, 0), (3, 5, 701, 128, 128),
    (2, 4, 1023, 64, 5), (2, 4, 1025, 64, 5), (1, 8, 4096, 64, 7), (1, 8, 4097, 256, 128), (1, 8, 5120, 128, 128), (1, 8, 5121, 128, 128),   # 32 segments, 40, 40, 48
    (8, 5, 64, 128, 8), (8, 5, 1, 64, 0), (4, 5, 3, 128, 1), (41, 1, 70, 128, 1),
])
def test_mask_and_gather(B, H, T, D, w):
    scores = synth.make_scores(B, H, T, seed=T + B, ties=True)
    scores[0, 0, T // 2] = float("nan")
    rng = np.random.default_rng(T)
    seq_lens = rng.integers(0, T + 1, B).astype(np.int32)
    seq_lens[0], seq_lens[-1] = T, min(T, 1)
    sl = torch.from_numpy(seq_lens).to(DEV)
    bits = torch.randint(-32768, 32768, (2, B, H, T, D), dtype=torch.int16)
    K, V = bits.view(torch.bfloat16)
    S64 = scores.double().numpy()
    idx, n, off, Ko, Vo = binding.kvzap_mask_compact(scores.to(DEV), 0.25, w, K.to(DEV), V.to(DEV), sl)
    parity.assert_prune_matches(idx, n, off, Ko, Vo, K, V, S64, 0.25, w, seq_lens)
    tau = torch.linspace(-1.0, 1.0, B * H).view(B, H)
    idx, n, off = binding.kvzap_mask_per_head(scores.to(DEV), tau.to(DEV), w, sl)
    ref = O.prune(S64, tau.double().numpy(), w, None, None, seq_lens)
    np.testing.assert_array_equal(parity.to_np(off), ref.offsets)
    np.testing.assert_array_equal(parity.to_np(n), ref.lengths)
    want = np.concatenate([i for row in ref.idx for i in row])
    np.testing.assert_array_equal(parity.to_np(idx)[:len(want)], want)


def test_gather_stops_at_the_capacity():
    s = torch.ones((1, 2, 300), device=DEV)
    K = torch.randn((1, 2, 300, 128)).bfloat16().to(DEV)
    out = [torch.zeros((400, 128), dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    binding.kvzap_mask_compact(s, 0.0, 4, K, K, K_out=out[0], V_out=out[1], cap_rows=350)
    for o in out:
        assert torch.equal(o[:350], K.view(600, 128)[:350]) and not o[350:].any()


def test_threshold_of_many_groups():
    # groups of more than 49152 scores: 24 of them and more are selected in one launch, fewer by the chain
    rng = np.random.default_rng(3)
    S = (rng.standard_normal((1, 24, 49153)) * 0.5 - 9).astype(np.float32)
    for heads in (23, 24):
        tau = binding.kvzap_topk_threshold(torch.from_numpy(S[:, :heads].copy()).to(DEV), 128, 20000, False)
        want = O.topk_threshold(S[:, :heads].astype(np.float64), 128, 20000, False, None)
        np.testing.assert_array_equal(parity.to_np(tau).astype(np.float64), want)


@pytest.mark.parametrize("pool", [1, 1023, 8192, 8193, 16384, 16385, 32769, 49152, 49153, 65536, 65537])
@pytest.mark.parametrize("heads", [1, 3])
def test_threshold(pool, heads):
    # `heads` pooled heads (per layer) that hold `pool` scores or just fewer, and one head of them
    T = max(1, pool // heads)
    rng = np.random.default_rng(pool + heads)
    S = rng.standard_normal((2, heads, T)).astype(np.float32)
    S[0, 0, :T // 5] = 0.5                                 # many ties
    S[1, 0, T // 2] = np.nan
    seq_lens = np.array([T, T // 3], np.int32)
    w = min(37, T // 2)
    for per_layer in (False, True):
        for k in (1, T // 7, T // 2, heads * (T - w) - 1, heads * T):
            tau = binding.kvzap_topk_threshold(torch.from_numpy(S).to(DEV), w, k, per_layer,
                                               torch.from_numpy(seq_lens).to(DEV))
            want = O.topk_threshold(S.astype(np.float64), w, k, per_layer, seq_lens)
            np.testing.assert_array_equal(parity.to_np(tau).astype(np.float64), want)


@pytest.mark.parametrize("heads,max_pages", [(1, 300), (255, 300), (256, 300), (257, 300), (1024, 300), (1025, 300),
                                             (1024, 512), (1024, 513), (32, 16384), (33, 16384), (3, 40000)])
def test_assign_pages(heads, max_pages):
    rng = np.random.default_rng(heads)
    lengths = rng.integers(0, 300, (1, heads)).astype(np.int32)
    free = rng.permutation(heads * 20).astype(np.int32)
    dev = [torch.from_numpy(a).to(DEV) for a in (lengths, free)]
    want, used, ok = O.assign_pages(lengths, 16, free, max_pages)
    table, res = binding.kvzap_assign_pages(dev[0], 16, dev[1], max_pages)
    assert ok and res[:2].tolist() == [used, 0]
    np.testing.assert_array_equal(parity.to_np(table), want)
    table, res = binding.kvzap_assign_pages(dev[0], 16, dev[1][:max(used - 1, 0)].clone(), max_pages)
    assert used == 0 or (res[:2].tolist() == [0, 1] and (parity.to_np(table) == -1).all())


# Every row of a chunk is loaded before its rank is known while the blocks are no more than the CUs: lengths
# around whole chunks, the last grid with that form and the first without, each row width, nothing and all
# kept, a capacity that ends inside a chunk
@pytest.mark.parametrize("B,H,T,D", [(1, 1, 1, 64), (1, 8, 127, 128), (2, 4, 129, 256), (3, 8, 701, 128), (1, 8, 4096, 64),
                                     (1, 8, 4097, 128), (1, 2, 16384, 256)])
@pytest.mark.parametrize("keep", [0.0, 0.4, 1.0])
def test_rows_loaded_ahead_of_their_ranks(B, H, T, D, keep):
    g = torch.Generator(device="cuda").manual_seed(T + D)
    scores = torch.rand((B, H, T), generator=g, device="cuda")
    K = torch.randn((B, H, T, D), generator=g, device="cuda").bfloat16()
    V = torch.randn((B, H, T, D), generator=g, device="cuda").bfloat16()
    seq = torch.tensor([T - 3 * b if T > 6 else T for b in range(B)], dtype=torch.int32, device="cuda")
    window, tau = (0 if keep == 0.0 else 5), 1.0 - keep if keep else 2.0
    t = torch.arange(T, device="cuda")
    n = seq.view(B, 1, 1)
    flags = (t < n) & ((t >= n - window) | (scores >= tau))
    total = int(flags.sum())
    for cap in {B * H * T, total // 2}:
        K_out = torch.full((B * H * T, D), -7.0, device="cuda").bfloat16()
        V_out = K_out.clone()
        idx, lengths, offsets, _, _ = binding.kvzap_mask_compact(scores, tau, window, K, V, seq, K_out=K_out, V_out=V_out, cap_rows=cap)
        assert torch.equal(lengths.view(B, H), flags.sum(-1).to(torch.int32)) and int(offsets[-1]) == total
        assert torch.equal(idx[:total], flags.nonzero()[:, 2].to(torch.int32))
        m = min(cap, total)
        assert torch.equal(K_out[:m], K[flags][:m]) and torch.equal(V_out[:m], V[flags][:m])
        assert (K_out[m:] == -7).all() and (V_out[m:] == -7).all()
