"""The work that a user of this library has it do, as measurable cases.

Five kinds of work, each through the public entry points of `paper_2601_07891_amd.binding`:

  compress  Algorithm 1 for one layer of a short prompt (score, then mask and gather into the
            engine's cache): what an interactive request pays per layer
  score     the surrogate's forward over a prompt: MLP with weights prepared at load time, MLP
            with raw weights, linear, and the MLP fused into the layer's input normalisation
  prune     threshold + window + gather on scores that are there: packed or paged output, one
            global threshold or a fixed budget per head or per layer
  decode    one decoding step of one layer: evict, then attend to the ragged cache, in
            contiguous slabs or in pages
  teacher   the scores that a surrogate is trained on, for one prompt

Shapes are those of this repository's own configurations (8 KV heads of 128, hidden size 4096
or 5120, MLP width an eighth of it, window 128) and neighbours of them.
"""
import math

import torch

from paper_2601_07891_amd import binding as kv

BF16 = torch.bfloat16
WINDOW = 128


def listed():
    return [
        # the smallest ordinary call: a 1k-token prompt with the linear surrogate
        dict(name="compress_1k_linear", kind="compress", scorer="linear", B=1, T=1024, Dh=4096, H=8,
             D=128, keep=0.5, ragged=False),
        # a few chat requests of different lengths, padded into one batch of an odd size
        dict(name="compress_3x701_mlp", kind="compress", scorer="mlp", B=3, T=701, Dh=4096, H=8,
             D=128, keep=0.5, ragged=True),
        # a document of a few thousand tokens, weights prepared when the model was loaded
        dict(name="score_7k", kind="score", scorer="mlp", entry="prepared", B=1, T=7001, Dh=4096,
             H=8, sigma=0.0),
        # the long-context layer that the benchmark is quoted on
        dict(name="score_128k", kind="score", scorer="mlp", entry="prepared", B=1, T=131072, Dh=4096,
             H=8, sigma=0.5),
        # a wider model, four long sequences at once: the largest scoring call
        dict(name="score_4x64k_wide", kind="score", scorer="mlp", entry="prepared", B=4, T=65536,
             Dh=5120, H=8, sigma=0.0),
        # the same batch with the linear surrogate: a pure read of the hidden states
        dict(name="score_4x64k_linear", kind="score", scorer="linear", entry="raw", B=4, T=65536,
             Dh=5120, H=8, sigma=0.0),
        # scorer and input normalisation in one, normalised states written for the projections;
        # a length that is no multiple of any tile
        dict(name="score_norm_30k", kind="score", scorer="mlp", entry="rmsnorm_states", B=1, T=30011,
             Dh=4096, H=8, sigma=0.5),
        # mask and gather of the long-context layer at 4x compression
        dict(name="prune_128k", kind="prune", select="threshold", page=0, B=1, T=131072, H=8, D=128,
             keep=0.25, ragged=False),
        # fixed budget per head into 16-row pages, three padded sequences of odd lengths
        dict(name="prune_topk_paged_3x20k", kind="prune", select="topk_head", page=16, B=3, T=20011,
             H=8, D=128, keep=0.3, ragged=True),
        # a full decoding batch over caches of 4k to 32k rows per head
        dict(name="decode_64", kind="decode", scorer="mlp", page=0, B=64, rows_lo=4096, rows_hi=32768,
             Dh=4096, H=8, HQ=32, keep=0.5),
        # a lightly loaded server: three sequences, paged cache, a few thousand rows
        dict(name="decode_3_paged", kind="decode", scorer="mlp", page=16, B=3, rows_lo=1024,
             rows_hi=8192, Dh=4096, H=8, HQ=32, keep=0.25),
        # training data: the scores of an 8k-token prompt against its own repetition
        dict(name="teacher_8k", kind="teacher", T=8192, Tq=8192, instr=32, H=8, HQ=32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["compress", "score", "score", "prune", "prune", "decode", "decode", "teacher"])
    if kind == "compress":
        B = rng.choice([1, 1, 2, 3, 4])
        return dict(kind=kind, scorer=rng.choice(["linear", "mlp"]), B=B, T=_log_int(rng, 160, 8192) // B + 1,
                    Dh=rng.choice([2048, 4096, 5120]), H=rng.choice([4, 8, 8]),
                    D=rng.choice([64, 128, 128, 128]), keep=round(rng.uniform(0.1, 0.75), 3),
                    ragged=B > 1 and rng.random() < 0.5)
    if kind == "score":
        entry = rng.choice(["prepared", "prepared", "raw", "linear", "rmsnorm", "rmsnorm_states"])
        B = rng.choice([1, 1, 2, 4])
        return dict(kind=kind, scorer="linear" if entry == "linear" else "mlp",
                    entry="raw" if entry == "linear" else entry, B=B,
                    T=_log_int(rng, 128, 131072) // B + 1, Dh=rng.choice([2048, 4096, 4096, 5120]),
                    H=rng.choice([4, 8, 8]), sigma=rng.choice([0.0, 0.5]))
    if kind == "prune":
        B = rng.choice([1, 1, 2, 3, 4])
        return dict(kind=kind, select=rng.choice(["threshold", "threshold", "topk_head", "topk_layer"]),
                    page=rng.choice([0, 0, 16, 64, 128]), B=B, T=_log_int(rng, 512, 131072) // B + 1,
                    H=rng.choice([4, 8, 8]), D=rng.choice([64, 128, 128, 256]),
                    keep=round(rng.uniform(0.1, 0.75), 3), ragged=B > 1 and rng.random() < 0.5)
    if kind == "decode":
        hi = _log_int(rng, 512, 32768)
        return dict(kind=kind, scorer=rng.choice(["mlp", "mlp", "mlp", "linear"]),
                    page=rng.choice([0, 0, 16, 64, 128]), B=_log_int(rng, 1, 64),
                    rows_lo=max(1, hi // rng.choice([1, 2, 8])), rows_hi=hi,
                    Dh=rng.choice([4096, 4096, 5120]), H=8, HQ=rng.choice([16, 32, 32, 64]),
                    keep=rng.choice([0.1, 0.25, 0.5]))
    T = _log_int(rng, 512, 8192)
    return dict(kind=kind, T=T, Tq=max(64, T // rng.choice([1, 1, 4])), instr=rng.choice([16, 32, 57]),
                H=8, HQ=rng.choice([16, 32]))


# ---- inputs -----------------------------------------------------------------------------

def _randn(g, shape, scale=1.0):
    out = torch.empty(shape, dtype=BF16, device=g.device)
    flat, step = out.view(-1), 1 << 28          # in pieces: the fp32 draws of a 5 GB cache stay small
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=g, device=g.device).mul_(scale)
    return out


def _weights(g, case):
    Dh, H = case["Dh"], case["H"]
    if case["scorer"] == "linear":
        return dict(W1=_randn(g, (H, Dh), Dh ** -0.5), b1=_randn(g, (H,), 0.1), W2=None, b2=None)
    M = Dh // 8
    return dict(W1=_randn(g, (M, Dh), Dh ** -0.5), b1=_randn(g, (M,), 0.1),
                W2=_randn(g, (H, M), M ** -0.5), b2=_randn(g, (H,), 0.1))


def _hidden(g, B, T, Dh, sigma=0.0):
    h = _randn(g, (B, T, Dh))
    if sigma > 0:                               # token scales of a real residual stream differ
        z = torch.exp(sigma * torch.randn((B, T, 1), generator=g, device=g.device)).to(BF16)
        for b in range(B):
            h[b].mul_(z[b])
    return h


def _seq_lens(g, case):
    if not case["ragged"]:
        return None
    B, T = case["B"], case["T"]
    n = torch.linspace(T / 2, T, B, device=g.device).round()
    return n[torch.randperm(B, generator=g, device=g.device)].to(torch.int32)


def _visible(case, seq_lens):
    """(position exists, position is protected by the window), each [B, 1, T]."""
    B, T = case["B"], case["T"]
    t = torch.arange(T, device="cuda")
    n = seq_lens if seq_lens is not None else torch.full((B,), T, device="cuda")
    n = n.long().view(B, 1, 1)
    return t < n, (t < n) & (t >= n - WINDOW)


def _plain_scores(hidden, w):
    x = hidden.float()
    z = x @ w["W1"].float().t()
    if w["b1"] is not None:
        z = z + w["b1"].float()
    if w["W2"] is not None:
        z = torch.nn.functional.gelu(z) @ w["W2"].float().t() + w["b2"].float()
    return z.transpose(1, 2).contiguous()


def _tau_in_a_gap(values, keep):
    """A threshold near the wanted quantile, in the middle of the widest gap between scores
    there: the kept set is then the same for every correct rounding of the scores."""
    v = values.sort().values
    n = v.numel()
    mid, half = int((1 - keep) * n), max(8, n // 10)
    v = v[max(0, mid - half):min(n, mid + half)].double()
    if v.numel() < 2:
        return 0.0
    i = int((v[1:] - v[:-1]).argmax())
    return float((v[i] + v[i + 1]) / 2)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + 17)
    return {"compress": _prepare_compress, "score": _prepare_score, "prune": _prepare_prune,
            "decode": _prepare_decode, "teacher": _prepare_teacher}[case["kind"]](case, g)


def _prepare_compress(case, g):
    B, T, H, D = (case[k] for k in "BTHD")
    s = dict(kind="compress", w=_weights(g, case), hidden=_hidden(g, B, T, case["Dh"]),
             K=_randn(g, (B, H, T, D)), V=_randn(g, (B, H, T, D)), seq_lens=_seq_lens(g, case))
    scores = _plain_scores(s["hidden"], s["w"])
    exists, window = _visible(case, s["seq_lens"])
    s["tau"] = _tau_in_a_gap(scores[(exists & ~window).expand(B, H, T)], case["keep"])
    _packed_cache(s, B * H * T, D)
    return s


def _packed_cache(s, rows, D):
    """The cache that the rows go to, as an engine owns it: as large as the prompt."""
    s["keep_idx"] = torch.zeros(rows, dtype=torch.int32, device="cuda")
    s["K_out"] = torch.zeros((rows, D), dtype=BF16, device="cuda")
    s["V_out"] = torch.zeros((rows, D), dtype=BF16, device="cuda")


def _prepare_score(case, g):
    s = dict(kind="score", entry=case["entry"], w=_weights(g, case),
             hidden=_hidden(g, case["B"], case["T"], case["Dh"], case["sigma"]))
    if case["entry"] == "prepared":
        s["W1p"] = kv.kvzap_prepare_scorer(s["w"]["W1"])
    elif case["entry"].startswith("rmsnorm"):
        s["gain"] = (1 + 0.1 * torch.randn(case["Dh"], generator=g, device="cuda")).to(BF16)
        s["W1p"] = kv.kvzap_prepare_scorer_rmsnorm(s["w"]["W1"], s["gain"])
    return s


def _prepare_prune(case, g):
    B, T, H, D = (case[k] for k in "BTHD")
    s = dict(kind="prune", select=case["select"], page=case["page"], seq_lens=_seq_lens(g, case),
             K=_randn(g, (B, H, T, D)), V=_randn(g, (B, H, T, D)))
    # heads differ in level and spread, so that their kept lengths do
    level = 0.5 * torch.randn((B, H, 1), generator=g, device="cuda")
    spread = torch.exp(0.3 * torch.randn((B, H, 1), generator=g, device="cuda"))
    s["scores"] = torch.randn((B, H, T), generator=g, device="cuda") * spread + level
    exists, window = _visible(case, s["seq_lens"])
    pool = s["scores"][(exists & ~window).expand(B, H, T)]
    if case["select"] == "threshold":
        k = max(1, min(pool.numel(), int((1 - case["keep"]) * pool.numel())))
        s["tau"] = float(pool.kthvalue(k).values) if pool.numel() else 0.0
    else:
        s["k"] = max(1, int(case["keep"] * max(1, T - WINDOW))) * (H if case["select"] == "topk_layer" else 1)
    _packed_cache(s, B * H * T, D)
    if case["page"]:
        P = case["page"]
        per_head = (T + P - 1) // P
        pages = B * H * per_head
        s["free"] = torch.randperm(pages, generator=g, device="cuda").to(torch.int32)
        s["max_pages"] = per_head
        s["K_out"] = torch.zeros((pages, P, D), dtype=BF16, device="cuda")
        s["V_out"] = torch.zeros((pages, P, D), dtype=BF16, device="cuda")
    return s


_ROOM = 6144           # rows that a cache can grow by: more than a long run of steps appends
_TOKENS = 16           # different new tokens, taken in turn


def _prepare_decode(case, g):
    B, H, HQ, P, Dh = case["B"], case["H"], case["HQ"], case["page"], case["Dh"]
    D = 128
    lengths = torch.linspace(case["rows_lo"], case["rows_hi"], B * H, device="cuda").round().long()
    lengths = lengths[torch.randperm(B * H, generator=g, device="cuda")].view(B, H)
    cap = lengths + _ROOM
    if P:
        counts = (cap.reshape(-1) + P - 1) // P
        total = int(counts.sum())
        st = kv.PagedDecodeState(B, H, D, WINDOW, P, total, int(counts.max()), "cuda")
        perm = torch.randperm(total, generator=g, device="cuda").to(torch.int32)
        first = torch.cumsum(counts, 0) - counts
        column = torch.arange(st.max_pages, device="cuda")
        st.block_table = torch.where(column < counts[:, None], perm[(first[:, None] + column).clamp(max=total - 1)],
                                     torch.tensor(-1, dtype=torch.int32, device="cuda")).contiguous()
        st.page_counts = counts.to(torch.int32).view(B, H)
        st.K_pool.copy_(_randn(g, st.K_pool.shape))
        st.V_pool.copy_(_randn(g, st.V_pool.shape))
    else:
        st = kv.DecodeState(B, H, D, WINDOW, cap.cpu(), "cuda")
        st.K_prefix.copy_(_randn(g, st.K_prefix.shape))
        st.V_prefix.copy_(_randn(g, st.V_prefix.shape))
    st.lengths.copy_(lengths)
    st.seq_pos.fill_(4 * case["rows_hi"] + 5)
    st.K_ring.copy_(_randn(g, st.K_ring.shape))
    st.V_ring.copy_(_randn(g, st.V_ring.shape))
    level = 0.65 if case["scorer"] == "mlp" else 1.0     # spread of the surrogate's scores
    st.score_ring.copy_(level * torch.randn(st.score_ring.shape, generator=g, device="cuda"))
    s = dict(kind="decode", page=P, st=st, w=_weights(g, case), at=0, max_rows=int(cap.max()),
             tau=level * float(torch.special.ndtri(torch.tensor(1.0 - case["keep"], dtype=torch.float64))),
             hidden=[_hidden(g, 1, B, Dh)[0].contiguous() for _ in range(_TOKENS)],
             k=[_randn(g, (B, H, D)) for _ in range(_TOKENS)],
             v=[_randn(g, (B, H, D)) for _ in range(_TOKENS)],
             q=[_randn(g, (B, HQ, D)) for _ in range(_TOKENS)])
    M = case["Dh"] // 8 if case["scorer"] == "mlp" else 0
    need = max(kv.kvzap_workspace_bytes(kv.CALL_DECODE_EVICT, B, 1, Dh, M, H),
               kv.kvzap_workspace_bytes(kv.CALL_ATTEND_DECODE, B, s["max_rows"], HQ, WINDOW, H), 256)
    s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")   # a serving loop keeps its scratch
    return s


def _prepare_teacher(case, g):
    H, HQ, T, Tq = (case[k] for k in ("H", "HQ", "T", "Tq"))
    return dict(kind="teacher", T=T, q=_randn(g, (HQ, Tq, 128)), k=_randn(g, (H, T + case["instr"] + Tq, 128)),
                vnorm=torch.rand((H, T), generator=g, device="cuda") * 3.0 + 0.1,
                hnorm=torch.rand((Tq,), generator=g, device="cuda") * 5.0 + 0.5)


# ---- one pass ---------------------------------------------------------------------------

def run(s):
    kind = s["kind"]
    if kind == "compress":
        w = s["w"]
        scores = kv.kvzap_score(s["hidden"], w["W1"], w["b1"], w["W2"], w["b2"])
        return scores, kv.kvzap_mask_compact(scores, s["tau"], WINDOW, s["K"], s["V"], s["seq_lens"],
                                             keep_idx=s["keep_idx"], K_out=s["K_out"], V_out=s["V_out"])
    if kind == "score":
        w, entry = s["w"], s["entry"]
        if entry == "raw":
            return kv.kvzap_score(s["hidden"], w["W1"], w["b1"], w["W2"], w["b2"])
        if entry == "prepared":
            return kv.kvzap_score_prepared(s["hidden"], s["W1p"], w["b1"], w["W2"], w["b2"])
        return kv.kvzap_score_rmsnorm(s["hidden"], s["W1p"], s["gain"], 1e-6, w["b1"], w["W2"], w["b2"],
                                      want_normed=entry == "rmsnorm_states")
    if kind == "prune":
        return _run_prune(s)
    if kind == "decode":
        return _run_decode(s)
    return kv.kvzap_teacher_scores(s["q"], s["k"], s["T"], 128 ** -0.5, s["vnorm"], s["hnorm"])


def _run_prune(s):
    scores, K, V = s["scores"], s["K"], s["V"]
    if s["select"] == "threshold" and not s["page"]:
        return kv.kvzap_mask_compact(scores, s["tau"], WINDOW, K, V, s["seq_lens"], keep_idx=s["keep_idx"],
                                     K_out=s["K_out"], V_out=s["V_out"])
    if s["select"] == "threshold":
        idx, lengths, offsets = kv.kvzap_mask(scores, s["tau"], WINDOW, s["seq_lens"], keep_idx=s["keep_idx"])
    else:
        tau = kv.kvzap_topk_threshold(scores, WINDOW, s["k"], s["select"] == "topk_layer", s["seq_lens"])
        idx, lengths, offsets = kv.kvzap_mask_per_head(scores, tau, WINDOW, s["seq_lens"], keep_idx=s["keep_idx"])
    if not s["page"]:
        K_out, V_out = kv.kvzap_compact(K, V, idx, lengths, offsets, s["K_out"], s["V_out"])
        return idx, lengths, offsets, K_out, V_out
    table, taken = kv.kvzap_assign_pages(lengths, s["page"], s["free"], s["max_pages"])
    kv.kvzap_compact_paged(K, V, idx, lengths, offsets, table, s["page"], s["K_out"], s["V_out"])
    return idx, lengths, offsets, table, taken[:2], s["K_out"], s["V_out"]


def _run_decode(s):
    st, w, i = s["st"], s["w"], s["at"]
    s["at"] = (i + 1) % _TOKENS
    scale = 128 ** -0.5
    if s["page"]:
        kv.kvzap_decode_evict_paged(s["hidden"][i], w["W1"], w["b1"], w["W2"], w["b2"], s["k"][i], s["v"][i],
                                    st, s["tau"], s["ws"])
        out = kv.kvzap_attend_decode_paged(s["q"][i], st.K_pool, st.V_pool, st.block_table, s["page"],
                                           st.lengths, st.K_ring, st.V_ring, st.seq_pos, WINDOW,
                                           s["max_rows"], scale, workspace=s["ws"])
        rows, where = (st.K_pool, st.V_pool), st.pos_pool
    else:
        kv.kvzap_decode_evict(s["hidden"][i], w["W1"], w["b1"], w["W2"], w["b2"], s["k"][i], s["v"][i],
                              st, s["tau"], s["ws"])
        out = kv.kvzap_attend_decode(s["q"][i], st.K_prefix, st.V_prefix, st.slab_offsets, st.lengths,
                                     st.K_ring, st.V_ring, st.seq_pos, WINDOW, s["max_rows"], scale,
                                     workspace=s["ws"])
        rows, where = (st.K_prefix, st.V_prefix), st.prefix_pos
    return out, rows, where, st.K_ring, st.V_ring, st.score_ring, st.lengths, st.seq_pos, st.error_flag


# ---- what a pass cannot do without ------------------------------------------------------

def _score_work(case, rows):
    Dh, H = case["Dh"], case["H"]
    if case["scorer"] == "linear":
        return 2 * rows * Dh + 2 * H * Dh + 4 * H * rows, 2.0 * rows * Dh * H
    M = Dh // 8
    return 2 * rows * Dh + 2 * M * (Dh + H) + 4 * H * rows, 2.0 * rows * M * (Dh + H)


def _prune_work(case):
    B, T, H, D = (case[k] for k in "BTHD")
    rows = B * H * T * (0.75 if case["ragged"] else 1.0)
    if case.get("select", "threshold") == "topk_layer" or case["keep"] >= 1:
        kept = min(rows, case["keep"] * rows)
    else:
        kept = min(rows, case["keep"] * rows + B * H * WINDOW * (1 - case["keep"]))
    return 4 * rows + kept * (4 + 8 * D)


def work(case):
    kind = case["kind"]
    if kind == "compress":
        b, f = _score_work(case, case["B"] * case["T"])
        return {"bytes": b + _prune_work(case), "flops": f}
    if kind == "score":
        b, f = _score_work(case, case["B"] * case["T"])
        if case["entry"].startswith("rmsnorm"):
            b += 4 * case["B"] * case["T"] + (2 * case["B"] * case["T"] * case["Dh"]
                                              if case["entry"] == "rmsnorm_states" else 0)
        return {"bytes": b, "flops": f}
    if kind == "prune":
        return {"bytes": _prune_work(case), "flops": 0}
    if kind == "decode":
        b, f = _score_work(case, case["B"])
        heads = case["B"] * case["H"]
        rows = heads * ((case["rows_lo"] + case["rows_hi"]) / 2 + WINDOW)
        # cache rows read once; q in, out written; the new pair in, the leaving pair moved
        b += rows * 512 + case["B"] * case["HQ"] * 512 + heads * 1024 * (1 + case["keep"])
        return {"bytes": b, "flops": f + rows * 512.0 * case["HQ"] / case["H"]}
    T, Tq, H, HQ = (case[k] for k in ("T", "Tq", "H", "HQ"))
    P0 = T + case["instr"]
    pairs = HQ * (Tq * P0 + Tq * (Tq + 1) / 2)
    return {"bytes": 256 * (HQ * Tq + H * (P0 + Tq)) + 8 * H * T + 4 * Tq, "flops": 256.0 * pairs}


def tolerance(case):
    """Floating results against another order of summation or another allowed rounding: about
    four times what the path differs by from itself in 64 bits."""
    kind = case["kind"]
    if kind == "prune":
        return "exact"                     # given scores: one result is right, byte for byte
    if kind == "decode":                   # bf16 output, bf16 softmax weights: 2.3e-3, 5.7e-3
        return {"rel": 8e-3, "max": 2.5e-2}
    if kind == "teacher":                  # fp32 logits and statistics: 1.9e-7, 7e-7
        return {"rel": 1e-6, "max": 5e-6}
    if case["scorer"] == "linear":         # fp32 sums over the hidden size: 4.4e-7, 3.7e-6
        return {"rel": 2e-6, "max": 2e-5}
    if case.get("entry", "").startswith("rmsnorm"):   # bf16 weights times gain, bf16 states: 1.7e-3, 6.6e-3
        return {"rel": 6e-3, "max": 2.5e-2}
    return {"rel": 8e-4, "max": 8e-3}      # fp16 activations: 2.0e-4, 2.0e-3
