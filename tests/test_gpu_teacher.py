"""GPU parity of kvzap_teacher_scores (KVzip Eq. 1 / KVzip+ Eq. 3, log space) against the
float64 oracle.

Tolerance: the logits are bf16 x bf16 products (exact in fp32) accumulated over D = 128 in
fp32 (relative 1e-5 of sum |terms|, i.e. a few 1e-4 absolute on logits of size ~10), the
row statistics sum up to ~1e4 exponentials in fp32 (1e-4 relative -> 1e-4 in the log).  The
test bound on the log score is 2e-3 + 1e-4 * |ref|."""
import numpy as np
import pytest
import torch

from oracle import kvzap_oracle as O
from paper_2601_07891_amd import binding, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D = 128


def _inputs(H, G, T, instr, Tq, seed, gain=1.0):
    g = torch.Generator().manual_seed(seed)
    Tk = T + instr + Tq
    q = (torch.randn((H * G, Tq, D), generator=g) * gain).bfloat16()
    k = torch.randn((H, Tk, D), generator=g).bfloat16()
    vn = torch.rand((H, T), generator=g) * 3.0 + 0.1
    hn = torch.rand((Tq,), generator=g) * 5.0 + 0.5
    return q, k, vn, hn


def _check(H, G, T, instr, Tq, seed, gain=1.0, norms=True, scale=None):
    q, k, vn, hn = _inputs(H, G, T, instr, Tq, seed, gain)
    scale = D ** -0.5 if scale is None else scale
    got = binding.kvzap_teacher_scores(q.to(DEV), k.to(DEV), T, scale,
                                       vn.to(DEV) if norms else None, hn.to(DEV) if norms else None)
    torch.cuda.synchronize()
    ref = O.teacher_log_scores(synth.f64(q), synth.f64(k), scale, T,
                               vn.double().numpy() if norms else None,
                               hn.double().numpy() if norms else None)
    err = np.abs(got.double().cpu().numpy() - ref)
    bound = 2e-3 + 1e-4 * np.abs(ref)
    assert (err <= bound).all(), f"max err {err.max():.3e} (ref range {ref.min():.2f}..{ref.max():.2f})"
    return ref


def test_small_ragged_shapes():
    for (T, instr, Tq) in [(1, 0, 1), (5, 3, 5), (31, 1, 33), (32, 0, 32), (33, 7, 31), (130, 9, 127)]:
        _check(H=2, G=2, T=T, instr=instr, Tq=Tq, seed=T + Tq)


def test_several_tiles_splits_and_groups():
    _check(H=2, G=4, T=700, instr=25, Tq=700, seed=1)
    _check(H=3, G=1, T=520, instr=11, Tq=300, seed=2)          # fewer repeated tokens than prompt
    _check(H=1, G=8, T=260, instr=40, Tq=513, seed=3)


def test_the_benchmark_shape():
    # bench.py's --stage teacher shape: an 8192-token prompt, 32 instruction tokens, the prompt
    # repeated, 8 KV heads x 4 query heads -- query splits and the longest-block-first order in
    # play.  The oracle recomputes the first and the last KV head (a few seconds each).
    H, G, T, instr = 8, 4, 8192, 32
    q, k, vn, hn = _inputs(H, G, T, instr, T, seed=11)
    scale = D ** -0.5
    got = binding.kvzap_teacher_scores(q.to(DEV), k.to(DEV), T, scale, vn.to(DEV), hn.to(DEV))
    torch.cuda.synchronize()
    got = got.double().cpu().numpy()
    assert np.isfinite(got).all()
    for h in (0, H - 1):
        ref = O.teacher_log_scores(synth.f64(q[h * G:(h + 1) * G]), synth.f64(k[h:h + 1]), scale, T,
                                   vn[h:h + 1].double().numpy(), hn.double().numpy())
        err = np.abs(got[h:h + 1] - ref)
        assert (err <= 2e-3 + 1e-4 * np.abs(ref)).all(), (h, err.max())


def test_kvzip_without_norms_is_the_unit_norm_case():
    ref = _check(H=2, G=2, T=300, instr=10, Tq=300, seed=4, norms=False)
    assert (ref <= 1e-9).all()                                   # attention weights are <= 1


def test_peaked_attention_and_the_copy_pattern():
    _check(H=2, G=2, T=400, instr=16, Tq=400, seed=5, gain=6.0)   # logits ~ N(0, 36)
    # copy pattern: the repeated token's query is a multiple of its original key
    g = torch.Generator().manual_seed(6)
    T, instr = 300, 12
    k = torch.randn((1, T + instr + T, D), generator=g).bfloat16()
    q = (k[:, :T].float() * 3.0).bfloat16().repeat(2, 1, 1)       # two query heads, same pattern
    got = binding.kvzap_teacher_scores(q.to(DEV), k.to(DEV), T, 1.0)
    ref = O.teacher_log_scores(synth.f64(q), synth.f64(k), 1.0, T)
    assert (np.exp(ref) > 0.99).all()
    assert np.abs(got.double().cpu().numpy() - ref).max() <= 2e-3


def test_prompt_shorter_than_the_scored_prefix_and_empty():
    # only the first T positions are scored; T may be smaller than P0
    q, k, vn, hn = _inputs(2, 2, 200, 10, 200, 7)
    got = binding.kvzap_teacher_scores(q.to(DEV), k.to(DEV), 77, D ** -0.5, vn[:, :77].contiguous().to(DEV), hn.to(DEV))
    ref = O.teacher_log_scores(synth.f64(q), synth.f64(k), D ** -0.5, 77, vn[:, :77].double().numpy(),
                               hn.double().numpy())
    assert np.abs(got.double().cpu().numpy() - ref).max() <= 3e-3
    empty = binding.kvzap_teacher_scores(q.to(DEV), k.to(DEV), 0, D ** -0.5)
    assert tuple(empty.shape) == (2, 0)


def test_rejects_bad_arguments():
    L = binding.lib()
    q = torch.zeros((4, 8, D), dtype=torch.bfloat16, device=DEV)
    k = torch.zeros((2, 20, D), dtype=torch.bfloat16, device=DEV)
    out = torch.zeros((2, 8), dtype=torch.float32, device=DEV)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
    call = lambda **kw: L.kvzap_teacher_scores(
        q.data_ptr(), k.data_ptr(), None, None, 0.1, out.data_ptr(), kw.get("H", 2), kw.get("HQ", 4),
        8, kw.get("Tk", 20), kw.get("T", 8), kw.get("D", D), ws.data_ptr(), kw.get("ws", ws.numel()), None)
    assert call() == 0
    assert call(T=13) == -2          # scored prefix longer than what precedes the repeated prompt
    assert call(HQ=3) == -2
    assert call(Tk=7) == -2          # fewer keys than queries
    assert call(D=64) == -4
    assert call(ws=8) == -6
    torch.cuda.synchronize()


@pytest.mark.parametrize("H,HQ,longest,T", [(1, 4, 1071, 965), (8, 16, 515, 418), (8, 32, 2224, 1805), (8, 32, 8192, 4096)])
def test_a_workspace_of_the_longest_prompt_serves_the_others(H, HQ, longest, T):
    g = torch.Generator().manual_seed(T)
    q = torch.randn((HQ, T, 128), generator=g).bfloat16().to(DEV)
    k = torch.randn((H, 2 * T + 16, 128), generator=g).bfloat16().to(DEV)
    want = binding.kvzap_teacher_scores(q, k, T, 128 ** -0.5)
    n = binding.kvzap_workspace_bytes(binding.CALL_TEACHER_SCORES, 1, longest, HQ, longest, H)
    ws = torch.full((n + 8192,), 0xff, dtype=torch.uint8, device=DEV)
    got = binding.kvzap_teacher_scores(q, k, T, 128 ** -0.5, workspace=ws[:n])
    assert (ws[n:] == 0xff).all()
    # The softmax sums in another order: each is a chain of one addition per tile of 32 keys and 16
    # inside a tile, 2^-24 of the sum each at most, on both sides (log scores: absolute); and two
    # roundings of row biases of up to 32, 2^-20 each.
    assert (got - want).abs().max() <= 2 * (2 * T // 32 + 16) * 2.0 ** -24 + 2 * 2.0 ** -20
    with pytest.raises(binding.KvzapError):        # nothing but the queries' biases fits here
        binding.kvzap_teacher_scores(q, k, T, 128 ** -0.5, workspace=ws[:(HQ * T * 4 + 255) // 256 * 256])


@pytest.mark.parametrize("T,instr,Tq", [
    (96, 0, 63), (95, 1, 64), (127, 1, 65),       # the first query sees 3 whole key tiles, 3, and 4
    (128, 31, 255), (129, 32, 257),               # blocks of 256 kept rows: one short, one more
    (1, 0, 300), (600, 40, 33),                   # every tile on the diagonal; two query tiles
    (511, 1, 33), (512, 3, 290), (1290, 0, 257),  # one share of the keys, two, five
])
def test_edges_of_tiles_and_of_whole_visible_groups(T, instr, Tq):
    _check(H=3, G=2, T=T, instr=instr, Tq=Tq, seed=T + Tq)
    _check(H=1, G=1, T=T, instr=instr, Tq=Tq, seed=T + Tq + 1, gain=8.0)   # the reference moves often


# As many shares as the rules give: four key tiles in a share, fewer queries than one tile, one item a share;
# and the fewest, in the least workspace that is accepted
@pytest.mark.parametrize("H,G,T,Tq", [(8, 2, 511, 30), (8, 2, 512, 33), (8, 4, 1300, 64), (4, 1, 1025, 257), (8, 2, 640, 640)])
def test_shares_at_the_ends_of_their_range(H, G, T, Tq):
    q, k, vn, hn = _inputs(H, G, T, 16, Tq, seed=T)
    ref = O.teacher_log_scores(synth.f64(q), synth.f64(k), D ** -0.5, T, vn.double().numpy(), hn.double().numpy())
    least = (H * G * ((Tq + 31) // 32 * 32) * 4 + 255) // 256 * 256 + (H * T * 4 + 255) // 256 * 256
    full = binding.kvzap_workspace_bytes(binding.CALL_TEACHER_SCORES, 1, T, H * G, Tq, H)
    assert full >= least
    for n in (full, least):
        ws = torch.full((n + 4096,), 0xff, dtype=torch.uint8, device=DEV)
        got = binding.kvzap_teacher_scores(q.to(DEV), k.to(DEV), T, D ** -0.5, vn.to(DEV), hn.to(DEV), workspace=ws[:n])
        err = np.abs(got.double().cpu().numpy() - ref)
        assert (err <= 2e-3 + 1e-4 * np.abs(ref)).all(), err.max()
        assert (ws[n:] == 0xff).all()
