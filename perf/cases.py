"""What a user of this library has it do, as timed cases.

The library serves two stages.  At inference a video diffusion transformer calls the sparse attention of
one (timestep, layer) after the other: block-sparse heads, heads that run on anchor rows, or both in one
call.  Before that, once per model and resolution, a calibration stage takes dense forwards' q and k and
turns them into block masks (block energy, selection, votes) and into the list of spatially repetitive heads
(similarity score).  The cases below are these calls at the sizes of the repository's own benchmark and at
generic smaller ones; ``draw`` spreads over the same ranges.

Masks are synthetic stand-ins for calibrated ones: a band inside each frame, stripes at the same place of
other frames, sink columns and the diagonal, and a fixed number of kept blocks per head, unevenly spread over
the rows.  q and k carry a positional component, as activations do, so that attention is concentrated.
"""
import math

import numpy as np
import torch

import paper_2603_05503_amd as pkg

FORWARD, ATTENTION, MASKS, HEADS = "forward", "attention", "calibrate_masks", "detect_heads"

# kind       forward: one launch of the sparse forward with its options (element type, layout, log-sum-exp)
#            attention: one CalibAttention call (sparse heads and/or anchor-row heads of one key)
#            calibrate_masks: block energy -> selection at eps -> votes, of one prompt batch
#            detect_heads: spatial similarity scores of all heads
# frames/rows/cols  token grid of the video; text: tokens without a position behind it
# flagged    how many of the heads are repetitive and take the anchor-row path with `anchors` rows per frame
# layout     packed [B,H,N,D]; bnhd: views of [B,N,H,D]; fused: views of one projection output [B,N,3,H,D]
_DEFAULTS = dict(kind=ATTENTION, B=1, H=40, frames=21, rows=30, cols=52, text=0, D=128, block_q=128, block_k=128,
                 density=0.3, repeat=0.1, flagged=0, anchors=5, dtype="bf16", layout="packed", lse=False,
                 intervals=True, eps=0.9)


def _case(name=None, **kw):
    c = dict(_DEFAULTS, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: two heads of one 32 x 32 frame, where launch and latency are everything
        _case("tiny", kind=FORWARD, H=2, frames=1, rows=32, cols=32, D=64, block_q=64, block_k=64, density=0.445,
              repeat=0.125, intervals=False),
        # a small model: ragged length, half precision, [B,N,H,D] activations, log-sum-exp asked for
        _case("small_f16_lse", kind=FORWARD, B=2, H=6, frames=5, rows=23, cols=29, text=77, D=64, block_q=128,
              block_k=64, density=0.5, repeat=0.05, dtype="f16", layout="bnhd", lse=True),
        # a low-resolution clip of 8190 tokens: about one row of blocks per workgroup slot of the chip
        _case("clip_8k", H=12, rows=15, cols=26, density=0.35),
        # the two guidance branches of a mid-sized clip in one batch, with wide key blocks
        _case("guided_16k_bk192", kind=FORWARD, B=2, H=16, frames=13, rows=30, cols=42, block_k=192, density=0.25,
              repeat=0.0),
        # the headline: 480p shape, 30 % of the blocks kept, a tenth of the query blocks repeated
        _case("480p_sparse"),
        # the first, high-noise steps of a generation keep (nearly) everything
        _case("480p_dense", density=1.0, repeat=0.0),
        # the longest sequence of the benchmark: 75 600 tokens
        _case("720p_sparse", rows=45, cols=80, repeat=0.2),
        # joint video/text attention on slices of a fused projection; text blocks are kept whole
        _case("joint_text_fused", kind=FORWARD, H=24, frames=28, rows=30, cols=53, text=256, density=0.25, repeat=0.15,
              layout="fused"),
        # a key with both kinds of heads: 32 sparse ones, 8 on five anchor rows per frame
        _case("480p_mixed_heads", density=0.25, repeat=0.0, flagged=8),
        # the anchor-row scheme on its own, all heads, as in the paper's table
        _case("480p_anchor_rows", flagged=40),
        # calibration: masks of one prompt
        _case("480p_calibrate_masks", kind=MASKS),
        # calibration: which heads repeat themselves
        _case("480p_detect_heads", kind=HEADS, H=24),
    ]


def _tokens(c):
    return c["frames"] * c["rows"] * c["cols"] + c["text"]


def _spread(rng, lo, hi):
    """Log-uniform integer in [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice([FORWARD] * 4 + [ATTENTION] * 4 + [MASKS] * 2 + [HEADS])
    while True:
        c = _case(kind=kind, B=rng.choice([1, 1, 1, 2]), H=_spread(rng, 1, 40), frames=_spread(rng, 1, 28),
                  rows=rng.randint(12, 45), cols=rng.randint(16, 80), D=rng.choice([64, 128, 128, 128]),
                  density=round(math.exp(rng.uniform(math.log(0.12), 0.0)), 3), repeat=round(rng.uniform(0.0, 0.3), 3),
                  anchors=rng.randint(1, 6), eps=round(rng.uniform(0.8, 0.99), 3))
        c["text"] = rng.choice([0, 0, rng.randint(1, 256)])
        c["block_q"] = rng.choice([128, 128, 128, 64])
        c["block_k"] = rng.choice([128, 128, 64])
        if kind == FORWARD:
            if c["D"] == 128 and c["block_q"] == 128 and rng.random() < 0.4:
                c["block_k"] = rng.choice([96, 160, 192])
            c["dtype"] = rng.choice(["bf16", "bf16", "f16"])
            c["layout"] = rng.choice(["packed", "bnhd", "fused"])
            c["lse"] = rng.random() < 0.3
            c["intervals"] = rng.random() < 0.5
        elif kind == ATTENTION:
            c["flagged"] = rng.choice([0, rng.randint(0, c["H"])])
        elif kind == HEADS:
            c["text"] = 0
        n, w = _tokens(c), work(c)
        # no dearer than the listed ones; small blocks and D = 64 run at a lower rate
        dear = w["flops"] * (1.0 if c["D"] == 128 and c["block_q"] == 128 else 1.6)
        if 600 <= n <= 76000 and c["B"] * c["H"] * n * c["D"] <= 4e8 and dear <= (1.8e13 if kind != MASKS else 9e12):
            return c


# ---- inputs ------------------------------------------------------------------------------------------------
def _blocks(n, block):
    return -(-n // block)


def _place(c, block, device):
    """(frame, offset inside the frame) of every block's centre token, and which blocks touch text tokens."""
    n, per_frame, n_video = _tokens(c), c["rows"] * c["cols"], _tokens(c) - c["text"]
    nb = _blocks(n, block)
    i = torch.arange(nb, device=device)
    centre = torch.clamp(i * block + block // 2, max=n_video - 1)
    text = ((i + 1) * block > n_video) if c["text"] else torch.zeros(nb, dtype=torch.bool, device=device)
    return centre, centre // per_frame, centre % per_frame, text


def _mask_and_repeat(c, heads, seed):
    """Block mask uint8 [heads, nbq, nbk] with exactly round(density * nbq * nbk) kept blocks per head (text rows
    and columns on top), and the map of repeated query blocks int32 [heads, nbq]."""
    dev = "cuda"
    gen = torch.Generator(device=dev).manual_seed(seed)
    rng = np.random.default_rng(seed)
    cq, fq, oq, tq = _place(c, c["block_q"], dev)
    ck, fk, ok, tk = _place(c, c["block_k"], dev)
    nbq, nbk, per_frame = cq.numel(), ck.numel(), c["rows"] * c["cols"]
    dtok = (cq[:, None] - ck[None, :]).abs().float()
    doff = (oq[:, None] - ok[None, :]).abs().float()
    doff = torch.minimum(doff, per_frame - doff)
    dfr = (fq[:, None] - fk[None, :]).abs().float()
    same = fq[:, None] == fk[None, :]
    forced = (cq[:, None] // c["block_k"]) == torch.arange(nbk, device=dev)[None, :]
    forced[:, 0] = True
    keep = max(int(round(c["density"] * nbq * nbk)), 1)
    mask = torch.empty((heads, nbq, nbk), dtype=torch.uint8, device=dev)
    ones = torch.full_like(dtok, -math.inf)
    for h in range(heads):
        if keep >= nbq * nbk:
            mask[h] = 1
            continue
        w_band = c["block_k"] * math.exp(rng.uniform(0.0, math.log(6.0)))
        w_stripe = c["block_k"] * math.exp(rng.uniform(math.log(0.4), math.log(2.5)))
        phase, waves = rng.uniform(0.0, 2.0 * math.pi), rng.uniform(3.0, 9.0)
        temp = torch.exp(0.45 * math.sqrt(2.0) * torch.sin(phase + waves * 2.0 * math.pi / nbq *
                                                           torch.arange(nbq, device=dev, dtype=torch.float32)))
        score = torch.maximum(torch.where(same, -dtok / w_band, ones), -(doff / w_stripe + rng.uniform(0.02, 0.4) * dfr))
        score = score / temp[:, None] + 0.15 * torch.randn(nbq, nbk, device=dev, generator=gen)
        score[forced] = math.inf
        m = torch.zeros(nbq * nbk, dtype=torch.uint8, device=dev)
        m[torch.topk(score.reshape(-1), keep, sorted=False).indices] = 1
        mask[h] = m.reshape(nbq, nbk)
    mask[:, tq, :] = 1
    mask[:, :, tk] = 1
    repeat = np.full((heads, nbq), -1, dtype=np.int32)
    eligible = ~tq.cpu().numpy()
    eligible[nbq - 1] = False  # the last block may be a short one
    elig = np.flatnonzero(eligible)
    n_rep = min(int(round(c["repeat"] * nbq)), elig.size - 1)
    for h in range(heads):
        if n_rep > 0:
            rep = np.sort(rng.choice(elig, size=n_rep, replace=False))
            src = np.setdiff1d(elig, rep)
            at = np.searchsorted(src, rep)
            left, right = src[np.clip(at - 1, 0, src.size - 1)], src[np.clip(at, 0, src.size - 1)]
            repeat[h, rep] = np.where(np.abs(left - rep) <= np.abs(right - rep), left, right)
    return mask.cpu().numpy(), repeat


def _qkv(c, seed, with_v=True):
    """q, k[, v] of logical shape [B, H, N, D] in the case's layout; x = g + 0.4 U[position] W_head for q and k."""
    dev = "cuda"
    gen = torch.Generator(device=dev).manual_seed(seed)
    B, H, N, D = c["B"], c["H"], _tokens(c), c["D"]
    dtype = torch.bfloat16 if c["dtype"] == "bf16" else torch.float16
    t = torch.arange(N, device=dev)
    n_video, per_frame = N - c["text"], c["rows"] * c["cols"]
    tv = torch.clamp(t, max=n_video - 1)
    f, o = tv // per_frame, tv % per_frame
    ang = 2.0 * math.pi * torch.stack([f / c["frames"], o // c["cols"] / c["rows"], o % c["cols"] / c["cols"]], 1).float()
    code = torch.cat([torch.sin(ang), torch.cos(ang)], 1)
    code[t >= n_video] = 0.0
    n = 3 if with_v else 2
    if c["layout"] == "fused":
        whole = torch.empty((B, N, 3, H, D), dtype=dtype, device=dev)
        out = [whole[:, :, i].transpose(1, 2) for i in range(3)]
    elif c["layout"] == "bnhd":
        out = [torch.empty((B, N, H, D), dtype=dtype, device=dev).transpose(1, 2) for _ in range(n)]
    else:
        out = [torch.empty((B, H, N, D), dtype=dtype, device=dev) for _ in range(n)]
    for h in range(H):
        w = 0.4 * torch.randn(code.shape[1], D, device=dev, generator=gen)
        bias = code @ w
        for i in range(n):
            x = torch.randn(B, N, D, device=dev, generator=gen)
            out[i][:, h] = (x + bias if i < 2 else x).to(dtype)
    return out


def prepare(case, seed):
    c = dict(case)
    B, H, N, D, kind = c["B"], c["H"], _tokens(c), c["D"], c["kind"]
    state = dict(kind=kind, scale=1.0 / math.sqrt(D), case=c)
    if kind in (FORWARD, ATTENTION):
        state["q"], state["k"], state["v"] = _qkv(c, seed)
        if c["layout"] == "packed":
            state["out"] = torch.empty((B, H, N, D), dtype=state["q"].dtype, device="cuda")
        else:
            state["out"] = torch.empty((B, N, H, D), dtype=state["q"].dtype, device="cuda").transpose(1, 2)
        mask, repeat = _mask_and_repeat(c, H, seed + 1)
        if kind == FORWARD:
            hp = pkg.compile_pattern(mask, repeat, H, N, c["block_q"], c["block_k"])
            state["pattern"] = hp.to_device("cuda", intervals=c["intervals"])
            state["lse"] = torch.empty((B, H, N), dtype=torch.float32, device="cuda") if c["lse"] else None
        else:
            flagged = np.random.default_rng(seed + 2).permutation(H)[:c["flagged"]].tolist()
            attn = pkg.CalibAttention(H, N, D, c["block_q"], c["block_k"], (c["frames"], c["rows"], c["cols"]),
                                      c["anchors"], intervals=c["intervals"])
            attn.add("key", mask, flagged, repeat)
            state["attn"] = attn
    else:
        state["q"], state["k"] = _qkv(c, seed, with_v=False)
        if kind == MASKS:
            nbytes = pkg.block_energy_workspace_bytes(N, c["block_q"], c["block_k"])
            state["workspace"] = torch.empty(nbytes // 4, dtype=torch.float32, device="cuda")
        else:
            partner = pkg.anchor_partner(c["frames"], c["rows"], c["cols"], c["anchors"])
            state["partner"] = torch.from_numpy(partner).to("cuda")
            state["workspace"] = torch.empty((B, H, partner.size, 3), dtype=torch.float32, device="cuda")
    return state


def run(state):
    kind, c = state["kind"], state["case"]
    if kind == FORWARD:
        out = pkg.sparse_attn_fwd(state["q"], state["k"], state["v"], state["out"], state["pattern"], state["scale"],
                                  lse=state["lse"])
        return out if state["lse"] is None else (out, state["lse"])
    if kind == ATTENTION:
        return state["attn"](state["q"], state["k"], state["v"], state["out"], "key", state["scale"])
    if kind == MASKS:
        energy = pkg.block_energy(state["q"], state["k"], c["block_q"], c["block_k"], state["scale"],
                                  workspace=state["workspace"])
        masks = pkg.select_blocks_device(energy, c["eps"])
        counts = torch.zeros(masks.shape[1:], dtype=torch.int16, device=masks.device)
        for b in range(masks.shape[0]):
            pkg.vote_accumulate_device(masks[b], counts)
        return energy, masks, counts
    # the caller's workspace holds the per-token sums of products that the scores are made of
    score = pkg.spatial_similarity(state["q"], state["k"], state["partner"], c["cols"], state["scale"],
                                   workspace=state["workspace"])
    return score, state["workspace"]


# ---- what a pass cannot do without -----------------------------------------------------------------------------
def work(case):
    c = case
    B, H, N, D = c["B"], c["H"], _tokens(c), c["D"]
    tensor = 2.0 * B * H * N * D
    nbq, nbk = _blocks(N, c["block_q"]), _blocks(N, c["block_k"])
    if c["kind"] == MASKS:
        # S = Q K^T once; q, k in, energies, mask and counters out
        return {"bytes": 2 * tensor + H * nbq * nbk * (5.0 * B + 2.0), "flops": 2.0 * B * H * N * N * D}
    if c["kind"] == HEADS:
        # S = Q K^T of every token; its partner's row of S is another token's
        return {"bytes": 2 * tensor + 4.0 * N + 12.0 * B * H * N, "flops": 2.0 * B * H * N * N * D}
    n_video = N - c["text"]
    text = c["text"] / N
    density = min(1.0, c["density"] + (1.0 - c["density"]) * 2.0 * text)
    computed = (1.0 - c["repeat"]) * n_video + c["text"]
    sparse = H - c["flagged"]
    pairs = sparse * density * computed * N  # (query, key) pairs of the block-sparse heads
    queries = sparse * computed
    if c["flagged"]:
        n_q = c["frames"] * min(c["anchors"], c["rows"]) * c["cols"] + c["text"]
        pairs += c["flagged"] * float(n_q) * N
        queries += c["flagged"] * n_q
    kept = sparse * density * (1.0 - c["repeat"]) * nbq * nbk
    nbytes = B * (2.0 * D * queries + 3.0 * 2.0 * D * H * N + (4.0 * H * N if c["lse"] else 0.0)) + kept * 0.5
    return {"bytes": nbytes, "flops": 4.0 * B * pairs * D}


def tolerance(case):
    if case["kind"] in (FORWARD, ATTENTION):
        # one rounding of the probabilities and one of the result: against fp64 2.2e-3 (bf16) and 2.8e-4 (fp16)
        # are measured, between two schedules 2.5e-3 and 3.4e-4; the log-sum-exp is fp32 (2e-6)
        return {"rel": 8e-3 if case["dtype"] == "bf16" else 1.2e-3}
    if case["kind"] == MASKS:
        # energies are fp32 sums of fp32 exponentials (against fp64 1e-7 at 4000 tokens, more for longer sums); a
        # block whose running sum meets eps within their rounding may fall on either side
        return {"rel": 1e-5, "differ": 2e-4}
    return {"rel": 1e-5}  # fp32 sums of products of probabilities


# ---- the same outputs in 64 bits, plain torch ------------------------------------------------------------------------
_EXACT_LOGITS = 1.2e11  # (query, key) pairs that take some 20 s


def _attention64(q, k, v, scale, visible=None):
    """Softmax attention of fp64 queries [n, D] over all keys (or those visible [n, N]), and its log-sum-exp."""
    s = (q @ k.T) * scale
    if visible is not None:
        s = s.masked_fill(~visible, -math.inf)
    lse = torch.logsumexp(s, 1)
    return torch.exp(s - lse[:, None]) @ v, lse


def _anchor_tokens(c):
    """Of every token, the token whose query it takes: same frame and column, nearest of the anchor rows (rows under
    the centres of equal segments, the lower one on a tie); text tokens keep their own."""
    rows, cols, k = c["rows"], c["cols"], min(c["anchors"], c["rows"])
    anchor = torch.tensor([(2 * j + 1) * rows // (2 * k) for j in range(k)])
    row = torch.arange(rows)
    nearest = anchor[(row[:, None] - anchor[None, :]).abs().argmin(1)]  # argmin: the first of equals
    shift = ((nearest - row) * cols).repeat_interleave(cols).repeat(c["frames"])
    own = torch.arange(_tokens(c))
    own[:shift.numel()] += shift
    return own.cuda()


def exact(case, seed):
    c = dict(case)
    B, H, N, D, kind = c["B"], c["H"], _tokens(c), c["D"], c["kind"]
    if B * H * float(N) * N * (2.0 if kind == HEADS else 1.0) > _EXACT_LOGITS:
        return None
    scale, dev = 1.0 / math.sqrt(D), "cuda"
    step = max(1, int(1.2e8) // N)  # queries at a time
    if kind in (FORWARD, ATTENTION):
        q, k, v = _qkv(c, seed)
        mask, repeat = _mask_and_repeat(c, H, seed + 1)
        flagged = set()
        if kind == ATTENTION:
            flagged = set(np.random.default_rng(seed + 2).permutation(H)[:c["flagged"]].tolist())
        bq, key_block = c["block_q"], torch.arange(N, device=dev) // c["block_k"]
        out = torch.empty((B, H, N, D), dtype=torch.float64, device=dev)
        lse = torch.empty((B, H, N), dtype=torch.float64, device=dev)
        for b in range(B):
            for h in range(H):
                qh, kh, vh = (t[b, h].double() for t in (q, k, v))
                if h in flagged:
                    source = _anchor_tokens(c)
                    visible = None
                else:
                    visible = torch.from_numpy(mask[h]).to(dev).bool()
                    rep = torch.from_numpy(repeat[h]).to(dev).long()
                    t = torch.arange(N, device=dev)
                    source = torch.where(rep[t // bq] >= 0, rep[t // bq] * bq + t % bq, t)
                todo = torch.unique(source)
                for i in range(0, todo.numel(), step):
                    at = todo[i:i + step]
                    see = None if visible is None else visible[at // bq][:, key_block]
                    out[b, h, at], lse[b, h, at] = _attention64(qh[at], kh, vh, scale, see)
                out[b, h], lse[b, h] = out[b, h, source], lse[b, h, source]
        return (out, lse) if c["lse"] and kind == FORWARD else out
    q, k = _qkv(c, seed, with_v=False)
    nbq, nbk = _blocks(N, c["block_q"]), _blocks(N, c["block_k"])
    if kind == MASKS:
        row_block, key_block = torch.arange(N, device=dev) // c["block_q"], torch.arange(N, device=dev) // c["block_k"]
        energy = torch.zeros((B, H, nbq, nbk), dtype=torch.float64, device=dev)
        for b in range(B):
            for h in range(H):
                qh, kh = q[b, h].double(), k[b, h].double()
                for i in range(0, N, step):
                    p = torch.softmax((qh[i:i + step] @ kh.T) * scale, 1)
                    mass = torch.zeros((p.shape[0], nbk), dtype=torch.float64, device=dev).index_add_(1, key_block, p)
                    energy[b, h].index_add_(0, row_block[i:i + step], mass)
        energy /= torch.bincount(row_block).double()[:, None]
        return energy, None, None  # a block at the edge of eps has no one answer
    n_tok = N - c["text"]
    source = _anchor_tokens(c)[:n_tok]
    triples = torch.empty((B, H, n_tok, 3), dtype=torch.float64, device=dev)
    for b in range(B):
        for h in range(H):
            qh, kh = q[b, h].double(), k[b, h].double()
            for i in range(0, n_tok, step):
                p = torch.softmax((qh[i:min(i + step, n_tok)] @ kh.T) * scale, 1)
                pa = torch.softmax((qh[source[i:i + step]] @ kh.T) * scale, 1)
                triples[b, h, i:i + step] = torch.stack([(p * pa).sum(1), (p * p).sum(1), (pa * pa).sum(1)], 1)
    rows = triples.reshape(B, H, n_tok // c["cols"], c["cols"], 3).sum(3)
    return (rows[..., 0] / torch.sqrt(rows[..., 1] * rows[..., 2])).mean(2), triples
