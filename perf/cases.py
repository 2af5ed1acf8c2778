"""The work that a program using this framework has it do, as cases that can be timed and compared.

A case is a dict of plain values.  Its `kind` is the part of the path that one pass runs:

  decode   attention of one decode step over `layers` packed caches, called one after the other
  step     one decode step of a model: every layer appends the new token and attends (a captured HIP graph, replayed)
  prefill  window scores -> widths -> reorder + quantize, for one layer's keys and values
  whole    prefill and one decode step of one layer
  scores   window scores only (pooled, or the literal pairwise form on the matrix cores)
  restore  a packed cache back to 16-bit rows in memory

Sizes: `batch` sequences of `frames` video frames of `per_frame` tokens (+ `tail` tokens that fill no window), windows of
`window` tokens, `text` prompt tokens; `ragged` != 0 makes it the seed of the sequences' own lengths (from an eighth
of `frames` up), window sizes and width mixes.  `top` and `mid` are the percentages of windows at the top width and at 4 bits.
"""
import math
import random

import torch

from paper_2605_02262_amd import binding as W

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
I32 = dict(dtype=torch.int32)

# (query heads, KV heads, head_dim, embedding size) of the configurations
SMALL = dict(heads=14, kv_heads=2, head_dim=64, dim=896)
LARGE = dict(heads=28, kv_heads=4, head_dim=128, dim=3584)


def _case(kind, **more):
    c = dict(kind=kind, batch=1, frames=32, per_frame=196, tail=0, window=196, text=128, ragged=0, heads=28, kv_heads=4, head_dim=128, dim=3584,
             group=64, dtype="bf16", top=20, mid=50, top_bits=8, mode="quota", layers=1, pairwise=False, fixed=False)
    c.update(more)
    return c


def listed():
    return [
        # the smallest calls: the whole path over 8 windows of 16 tokens in fp32 (launches and host work are all there is)
        _case("whole", name="tiny_whole_f32", frames=8, per_frame=16, window=16, text=16, group=32, dtype="f32", top=25, **SMALL),
        # a short clip in a small model, one request: one layer's decode call (latency)
        _case("decode", name="small_decode_b1", group=32, top=25, **SMALL),
        # one request of 100 frames with windows of 32 and a 16-bit top tier: a decode step of all layers as a serving loop replays it
        _case("step", name="paper_tiers_step", frames=100, window=32, text=135, top=0.4, mid=35, top_bits=16, layers=28, **LARGE),
        # eight requests of 64 frames: a decode step of all layers
        _case("step", name="batch8_step", batch=8, frames=64, text=256, layers=28, **LARGE),
        # four long videos: decode attention, one layer after the other
        _case("decode", name="long_decode", batch=4, frames=256, text=512, top=10, mid=40, layers=4, **LARGE),
        # a serving batch of 32 requests of very different lengths
        _case("decode", name="ragged_decode", batch=32, frames=128, text=256, ragged=4077, layers=2, **LARGE),
        # finer groups (four per head): lower error for a little more metadata
        _case("decode", name="group32_decode", batch=8, frames=64, text=251, group=32, layers=2, **LARGE),
        # one group per head of a small model with an fp16 cache, odd lengths
        _case("decode", name="group64_f16_decode", batch=16, frames=33, text=77, tail=13, group=64, dtype="f16", layers=2, **SMALL),
        # prefill of the four long videos
        _case("prefill", name="long_prefill", batch=4, frames=256, text=512, top=10, mid=40, **LARGE),
        # prefill of a ragged fp16 batch, widths by thresholds
        _case("prefill", name="ragged_prefill_f16", batch=16, frames=96, text=201, tail=31, ragged=91, dtype="f16", mode="threshold", **LARGE),
        # scoring by the literal pairwise form
        _case("scores", name="pairwise_scores", batch=8, frames=64, text=256, pairwise=True, **LARGE),
        # a batch of caches dequantized to memory
        _case("restore", name="batch8_restore", batch=8, frames=64, text=256, **LARGE),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = max(_cost(c) for c in listed())
    kind = rng.choice(["decode", "decode", "decode", "step", "prefill", "prefill", "whole", "scores", "restore"])
    model = dict(rng.choice([SMALL, LARGE, LARGE, dict(heads=32, kv_heads=8, head_dim=128, dim=4096), dict(heads=8, kv_heads=8, head_dim=64, dim=512)]))
    hd = model["head_dim"]
    c = _case(kind, **model)
    c["group"] = rng.choice([hd // 2, hd // 2, hd // 2, hd, 32])
    c["dtype"] = rng.choice(["bf16", "bf16", "bf16", "f16"])
    if kind in ("prefill", "whole") and rng.random() < 0.15:
        c["dtype"] = "f32"
    c["window"] = rng.choice([16, 32, 98, 196, 196])
    c["per_frame"] = rng.choice([16, 144, 196, 196])
    c["tail"] = rng.choice([0, 0, rng.randrange(c["window"])])
    c["batch"] = _log(rng, 1, 32)
    tokens = _log(rng, 8 * c["window"], 250000 if kind != "whole" else 20000)     # of the whole batch
    tokens = min(tokens, 3900 * c["window"] * c["batch"])                         # (a sequence has at most 8192 windows)
    c["frames"] = max(1, -(-tokens // (c["batch"] * c["per_frame"])), -(-2 * c["window"] // c["per_frame"]))
    c["text"] = _log(rng, 5, 600)
    c["top"] = rng.choice([0, 10, 20, 25, 50, 100])
    c["mid"] = rng.choice([m for m in (0, 20, 35, 40, 50) if m + c["top"] <= 100])
    c["top_bits"] = rng.choice([8, 8, 8, 16])
    c["mode"] = rng.choice(["quota", "quota", "threshold"]) if kind == "prefill" else "quota"
    if c["batch"] > 2 and rng.random() < 0.4:
        c["ragged"] = rng.randrange(1, 1 << 20)
    if kind == "decode":
        c["layers"] = rng.choice([1, 2, 4])
        c["fixed"] = rng.random() < 0.1
    if kind == "step":
        c["layers"] = rng.choice([4, 12, 28])
    if kind == "scores":
        c["pairwise"] = rng.random() < 0.6
    while _cost(c) > most:
        if c["frames"] > 1:
            c["frames"] = max(1, c["frames"] * 3 // 4)
        elif c["batch"] > 1:
            c["batch"] -= 1
        else:
            c["layers"] = 1
    return c


# ------------------------------------------------------------------------------------------------------------------------
# sizes
# ------------------------------------------------------------------------------------------------------------------------
class _Sizes:
    """The sequences of a case, and the tables that describe them to the framework (host lists)."""

    def __init__(self, c):
        rng = random.Random(c["ragged"]) if c["ragged"] else None
        self.win, self.windows, self.visual, self.text, self.quota = [], [], [], [], []
        for b in range(c["batch"]):
            frames, window, top, mid = c["frames"], c["window"], c["top"], c["mid"]
            if rng:
                frames = rng.randint(max(1, frames // 8), frames)
                window = rng.choice([window, max(16, window // 2)])
                cut = sorted(rng.uniform(0, 100) for _ in range(2))
                if c["mode"] == "quota":
                    top, mid = (0, 0) if b == 0 else (100, 0) if b == 1 else (cut[0], cut[1] - cut[0])
            visual = frames * c["per_frame"] + c["tail"]
            n = visual // window
            n_top, n_both = int(top * n / 100 + 0.5), int((top + mid) * n / 100 + 0.5)
            self.win.append(window)
            self.windows.append(n)
            self.visual.append(visual)
            self.text.append(c["text"])
            self.quota.append((n_top, n_both - n_top, n - n_both))
        add = lambda v: [sum(v[:i]) for i in range(len(v) + 1)]  # noqa: E731
        self.vis_off, self.txt_off, self.win_off = add(self.visual), add(self.text), add(self.windows)
        self.kv_off = add([v + t for v, t in zip(self.visual, self.text)])
        self.longest = max(v + t for v, t in zip(self.visual, self.text))
        self.most_windows = max(self.windows)
        self.pin = all(q[0] > 0 for q in self.quota)

    def tokens(self, c):
        """(2-bit, 4-bit, 8-bit, 16-bit) tokens of the batch."""
        n2 = sum(q[2] * w for q, w in zip(self.quota, self.win))
        n4 = sum(q[1] * w for q, w in zip(self.quota, self.win))
        n_top = sum(q[0] * w for q, w in zip(self.quota, self.win))
        rest = self.kv_off[-1] - n2 - n4 - n_top
        return (n2, n4, n_top, rest) if c["top_bits"] == 8 else (n2, n4, 0, rest + n_top)

    def capacities(self, c, slack):
        """Class capacities and first 16-bit rows: the quotas' own sizes, or room for every window where thresholds decide."""
        pad = lambda n: (n + 31) // 32 * 32  # noqa: E731
        cap, rows = [0, 0, 0], []
        for q, w, n, v, t in zip(self.quota, self.win, self.windows, self.visual, self.text):
            room = (n, n, n) if c["mode"] == "threshold" else (q[2], q[1], q[0])
            top16 = c["top_bits"] == 16
            for k in range(3):
                cap[k] += 0 if (k == 2 and top16) else pad(room[k] * w)
            rows.append((room[2] * w if top16 else 0) + v - n * w + t + slack)
        return cap, [sum(rows[:i]) for i in range(len(rows) + 1)]


def _packed_bytes(c, s):
    n = s.tokens(c)
    per = 2 * c["kv_heads"]
    hd, groups = c["head_dim"], c["head_dim"] // c["group"]
    return sum(t * per * (hd * b // 8 + 4 * groups) for t, b in zip(n[:3], (2, 4, 8))) + n[3] * per * hd * 2


def work(c):
    s = _Sizes(c)
    rows, size = s.kv_off[-1], 4 if c["dtype"] == "f32" else 2
    per_row = 2 * c["kv_heads"] * c["head_dim"]                                     # elements of a token's keys and values
    packed = _packed_bytes(c, s)
    emb = (s.vis_off[-1] + s.txt_off[-1]) * c["dim"] * size
    attend = dict(bytes=packed + c["batch"] * c["heads"] * c["head_dim"] * (size + 4), flops=4 * c["heads"] * c["head_dim"] * rows)
    if c["kind"] in ("decode", "step"):
        new = 2 * c["batch"] * per_row * 2 if c["kind"] == "step" else 0            # new rows read and written
        return dict(bytes=c["layers"] * (attend["bytes"] + new), flops=c["layers"] * attend["flops"])
    if c["kind"] == "restore":
        return dict(bytes=packed + rows * per_row * 2, flops=2 * rows * per_row)
    if c["kind"] == "scores":
        pairs = sum(v * t for v, t in zip(s.visual, s.text))
        return dict(bytes=emb, flops=2 * pairs * c["dim"] if c["pairwise"] else 4 * s.vis_off[-1] * c["dim"])
    pre = dict(bytes=emb + rows * per_row * size + packed, flops=4 * s.vis_off[-1] * c["dim"] + 4 * rows * per_row)
    if c["kind"] == "whole":
        return dict(bytes=pre["bytes"] + attend["bytes"], flops=pre["flops"] + attend["flops"])
    return pre


def _cost(c):
    w = work(c)
    return max(w["bytes"], w["flops"] / 50)


def tolerance(c):
    if c["kind"] == "restore":
        return "exact"
    if c["kind"] in ("prefill", "scores"):
        return {"rel": 3e-7, "max": 1e-6}        # fp32 sums of a few thousand terms (6e-8 against fp64); all that follows the scores is exact
    if c["head_dim"] == 2 * c["group"]:          # softmax weights meet the value scales in fp16: 1e-4..3e-4, single values up to 1.6e-3
        return {"rel": 1e-3, "max": 7e-3}
    return {"rel": 5e-5, "max": 5e-4}            # weights and sums of fp32 accuracy over a whole sequence


# ------------------------------------------------------------------------------------------------------------------------
# what a program has in hand
# ------------------------------------------------------------------------------------------------------------------------
class _State:
    pass


def prepare(c, seed):
    s, st = _Sizes(c), _State()
    gen = torch.Generator(device="cuda").manual_seed(seed)
    randn = lambda *shape: torch.randn(*shape, generator=gen, device="cuda")  # noqa: E731
    dt = DTYPES[c["dtype"]]
    dt16 = torch.bfloat16 if c["dtype"] == "bf16" else torch.float16
    B, Hq, Hkv, hd, L, D = c["batch"], c["heads"], c["kv_heads"], c["head_dim"], c["layers"], c["dim"]
    table = lambda v: torch.tensor(v, **I32).cuda()  # noqa: E731
    st.case, st.sizes, st.scale = c, s, 1.0 / math.sqrt(hd)
    st.vis_off, st.txt_off, st.win_off, st.kv_off = table(s.vis_off), table(s.txt_off), table(s.win_off), table(s.kv_off)
    st.win_size, st.quota = table(s.win), table([list(q) for q in s.quota])
    embeds = c["kind"] in ("prefill", "whole", "scores")

    # splits and workspace: what the framework picks for these lengths
    slack = 8 if c["kind"] == "step" else 0
    cap, off16 = s.capacities(c, slack)
    st.by_length = W.DECODE_BY_LENGTH if c["ragged"] else 0
    longest = s.longest + slack
    splits = W.auto_splits_ragged(B, Hkv, longest, sum(cap) + off16[-1]) if c["ragged"] else W.auto_splits(B, Hkv, longest)
    st.longest = longest
    st.ctx = W.Context(W.workspace_bytes(B, Hq, hd, splits, s.vis_off[-1] if embeds else 0, s.txt_off[-1] if embeds else 0, D if embeds else 0))
    st.algo = W.DECODE_AUTO | st.by_length | (W.DECODE_FIXED_SHARES if c["fixed"] else 0)

    if embeds:      # text ~ N(0, 1); a window's tokens are alpha_i u + N(0, I), u the direction of the mean text token
        st.text = torch.empty(s.txt_off[-1], D, dtype=dt, device="cuda")
        st.visual = torch.empty(s.vis_off[-1], D, dtype=dt, device="cuda")
        for b in range(B):
            t = randn(s.text[b], D)
            u = torch.nn.functional.normalize(t.mean(0), dim=0)
            alpha = torch.rand(s.windows[b], generator=gen, device="cuda").repeat_interleave(s.win[b])
            st.text[s.txt_off[b]:s.txt_off[b + 1]] = t.to(dt)
            for lo in range(0, s.visual[b], 16384):
                hi = min(s.visual[b], lo + 16384)
                v = randn(hi - lo, D)
                n = max(0, min(hi, alpha.numel()) - lo)
                v[:n].addcmul_(alpha[lo:lo + n, None], u[None, :])
                st.visual[s.vis_off[b] + lo:s.vis_off[b] + hi] = v.to(dt)
        # scores are about alpha / sqrt(text tokens x dim): thresholds that give the case's mix
        one = [1.0 / math.sqrt(t * D) for t in s.text]
        st.thresholds = torch.tensor([[x * (100 - c["top"] - c["mid"]) / 100, x * (100 - c["top"]) / 100] for x in one], device="cuda")
        if c["kind"] == "scores":
            return st

    # keys with channel outliers, values ~ N(0, 1), queries that give logits of standard deviation 2
    rep = Hq // Hkv
    st.caches, st.q = [], []
    for layer in range(L):
        outlier = torch.exp((1.0 if hd == 64 else 1.5) * randn(Hkv, hd))
        K = torch.empty(s.kv_off[-1], Hkv, hd, dtype=dt, device="cuda")
        V = torch.empty_like(K)
        for lo in range(0, s.kv_off[-1], 65536):
            hi = min(s.kv_off[-1], lo + 65536)
            K[lo:hi] = (randn(hi - lo, Hkv, hd) * outlier).to(dt)
            V[lo:hi] = randn(hi - lo, Hkv, hd).to(dt)
        q = randn(B, Hq, hd)
        dev = st.scale * (q.view(B, Hkv, rep, hd) * outlier[None, :, None]).square().sum(-1).sqrt().view(B, Hq, 1)
        st.q.append((q * (2.0 / dev)).to(dt))
        cache = W.PackedKV(B, Hkv, hd, c["group"], dt16, cap, off16, fill=0)
        st.caches.append(cache)
        if embeds:
            st.K, st.V = K, V
            continue
        scores = torch.rand(s.win_off[-1], generator=gen, device="cuda")
        _, perm, seg = W.wq_assign_bits(st.ctx, scores, st.win_off, s.most_windows, W.MODE_QUOTA, st.quota, None, c["top_bits"], int(s.pin))
        W.wq_reorder_quantize(st.ctx, K, V, st.kv_off, st.win_size, st.win_off, perm, seg, s.kv_off[-1], cache)
    st.out = torch.empty(L, B, Hq, hd, device="cuda")
    st.lse = torch.empty(L, B, Hq, device="cuda")
    if c["kind"] == "restore":
        rows = [0]
        for v, t in zip(s.visual, s.text):
            rows.append(rows[-1] + v + t)
        st.dense = W.PackedKV(B, Hkv, hd, c["group"], dt16, [0, 0, 0], rows)
    if c["kind"] == "step":
        st.k_new = [(randn(B, Hkv, hd) * 0.5).to(dt16) for _ in range(L)]
        st.v_new = [randn(B, Hkv, hd).to(dt16) for _ in range(L)]
        # the lengths of all layers' 16-bit segments in one table, so that one launch takes a step back to the prompt
        st.prompt_rows = torch.stack([k.len16 for k in st.caches])
        st.rows = st.prompt_rows.clone()
        for k, n in zip(st.caches, st.rows):
            k.len16 = n
            k.desc.len16 = n.data_ptr()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        st.graph = torch.cuda.CUDAGraph()
        st.ctx.set_stream(side)
        with torch.cuda.stream(side):
            _step(st)
            side.synchronize()
            with torch.cuda.graph(st.graph, stream=side):
                _step(st)
        torch.cuda.current_stream().wait_stream(side)
    return st


def _step(st):
    torch.add(st.prompt_rows, 0, out=st.rows)      # another continuation of the same prompt
    for layer, cache in enumerate(st.caches):
        W.wq_decode_append_attention(st.ctx, st.q[layer], cache, st.k_new[layer], st.v_new[layer], st.scale, 0, st.longest, st.algo, out=st.out[layer])


def _prefill(st):
    c, s, cache = st.case, st.sizes, st.caches[0]
    scores = W.wq_window_scores(st.ctx, st.visual, st.text, st.vis_off, st.txt_off, st.win_size, st.win_off, s.vis_off[-1], s.txt_off[-1], s.win_off[-1])
    if c["mode"] == "threshold":
        bits, perm, seg = W.wq_assign_bits(st.ctx, scores, st.win_off, s.most_windows, W.MODE_THRESHOLD, None, st.thresholds, c["top_bits"], 1)
    else:
        bits, perm, seg = W.wq_assign_bits(st.ctx, scores, st.win_off, s.most_windows, W.MODE_QUOTA, st.quota, None, c["top_bits"], int(s.pin))
    W.wq_reorder_quantize(st.ctx, st.K, st.V, st.kv_off, st.win_size, st.win_off, perm, seg, s.kv_off[-1], cache)
    return dict(scores=scores, bits=bits, perm=perm, seg=seg, codes=cache.codes, meta=cache.meta, off=cache.cls_off, len=cache.cls_len, k16=cache.k16,
                v16=cache.v16, len16=cache.len16, v_scale_max=cache.v_scale_max[:c["batch"]])


def _decode(st, layer):
    W.wq_decode_attention(st.ctx, st.q[layer], st.caches[layer], st.scale, 0, st.longest, st.algo, out=st.out[layer], lse=st.lse[layer])


def run(st):
    c, s = st.case, st.sizes
    if c["kind"] == "scores":
        return W.wq_window_scores(st.ctx, st.visual, st.text, st.vis_off, st.txt_off, st.win_size, st.win_off, s.vis_off[-1], s.txt_off[-1], s.win_off[-1],
                                  algo=W.SCORE_PAIRWISE_MFMA if c["pairwise"] else W.SCORE_AUTO)
    if c["kind"] == "step":
        st.graph.replay()
        return dict(out=st.out, rows=st.rows, k16=[k.k16 for k in st.caches], v16=[k.v16 for k in st.caches])
    if c["kind"] == "restore":
        W.wq_dequantize(st.ctx, st.caches[0], st.dense)
        return dict(k16=st.dense.k16, v16=st.dense.v16, len16=st.dense.len16)
    got = _prefill(st) if c["kind"] in ("prefill", "whole") else {}
    if c["kind"] in ("decode", "whole"):
        for layer in range(c["layers"]):
            _decode(st, layer)
        got.update(out=st.out, lse=st.lse)
    return got
