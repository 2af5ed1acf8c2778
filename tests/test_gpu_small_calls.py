"""Scoring and quantizing of a few windows in one launch each: the same bits as the launches of larger calls (needs an MI355X)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _table(v):
    return torch.tensor(v, dtype=torch.int32, device="cuda")


def _offsets(v):
    out = [0]
    for x in v:
        out.append(out[-1] + x)
    return out


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("dim", [8, 504, 896, 1544, 4096])
def test_scores_of_a_small_call(dim, dtype):
    """Windows of 1, 16, 17 and 64 rows, texts of 0, 1, 8, 9, 31 .. 65 tokens (slices of 32), a zero row; the same batch beside a
    sequence that has only text, more of it than the one-launch form takes."""
    from paper_2605_02262_amd import binding as W
    gen = torch.Generator(device="cuda").manual_seed(dim)
    size = torch.empty(0, dtype=dtype).element_size()
    for window, n_win, texts in ((16, [3, 0, 2], [16, 3, 0]), (1, [5, 2], [1, 8]), (17, [1, 2], [9, 7]), (64, [2], [6]), (64, [1], [33]), (17, [2, 1], [50, 51]), (3, [2, 1, 1], [32, 31, 65])):
        texts = [min(n, (128 << 10) // (dim * size * len(texts))) for n in texts]
        rows = [n * window + 2 for n in n_win]
        vis = torch.randn(sum(rows), dim, generator=gen, device="cuda").to(dtype)
        vis[1] = 0
        more = 300
        txt = torch.randn(sum(texts) + more, dim, generator=gen, device="cuda").to(dtype)
        got = []
        for extra in (False, True):
            r, t, n = (rows + [0], texts + [more], n_win + [0]) if extra else (rows, texts, n_win)
            ctx = W.Context(W.workspace_bytes(len(r), 0, 0, 0, sum(r), sum(t), dim))
            got.append(W.wq_window_scores(ctx, vis, txt[:sum(t)], _table(_offsets(r)), _table(_offsets(t)), _table([window] * len(r)),
                                          _table(_offsets(n)), sum(r), sum(t), sum(n)))
        assert torch.equal(got[0], got[1]), (window, texts)
        assert torch.isfinite(got[0]).all() and (max(texts) == 0 or got[0].abs().max() > 0)


@pytest.mark.parametrize("dtype,hd,group", [(torch.bfloat16, 128, 64), (torch.float16, 64, 64), (torch.float32, 128, 32)])
@pytest.mark.parametrize("short", [False, True], ids=["fits", "overflows"])
def test_quantizing_a_small_call(dtype, hd, group, short):
    """16 sequences (one launch) and the same with an empty 17th (three): every class empty somewhere, partial blocks, 16-bit
    windows, tails, and capacities that some sequences do not fit.  A context is used twice: its counter is zero again."""
    from paper_2605_02262_amd import binding as W
    gen = torch.Generator(device="cuda").manual_seed(hd + group)
    heads, win = 2, [5, 16, 32, 33, 1, 7, 16, 3, 40, 2, 31, 16, 9, 4, 8, 6]
    seg = [[(b + c) % 3 if b != 5 else 0 for c in range(4)] for b in range(16)]
    n_win = [sum(s) for s in seg]
    rows = [n * w + b % 4 for b, (n, w) in enumerate(zip(n_win, win))]
    K = torch.randn(sum(rows), heads, hd, generator=gen, device="cuda").to(dtype)
    V = torch.randn(sum(rows), heads, hd, generator=gen, device="cuda").to(dtype)
    perm = torch.cat([torch.randperm(n, generator=gen, device="cuda") for n in n_win]).to(torch.int32)
    pad = lambda n: (n + 31) // 32 * 32  # noqa: E731
    cap = [sum(pad(s[c] * w) for s, w in zip(seg, win)) for c in range(3)]
    n16 = [s[3] * w + r - n * w for s, w, r, n in zip(seg, win, rows, n_win)]
    if short:
        cap = [c - 32 for c in cap]
        n16[2] -= 1
    dt16 = torch.bfloat16 if dtype == torch.bfloat16 else torch.float16
    runs = []
    for extra in (0, 1, 0):
        B = 16 + extra
        ctx = runs[0][1] if len(runs) == 2 else W.Context(W.workspace_bytes(B))
        pk = W.PackedKV(B, heads, hd, group, dt16, cap, _offsets(n16 + [0] * extra), fill=0)
        W.wq_reorder_quantize(ctx, K, V, _table(_offsets(rows + [0] * extra)), _table(win + [1] * extra), _table(_offsets(n_win + [0] * extra)),
                              perm, _table(seg + [[0] * 4] * extra), sum(rows), pk)
        status = ctx.device_status()
        assert status == (W.DEV_CLASS_OVERFLOW | W.DEV_SEG16_OVERFLOW if short else 0)
        runs.append((pk, ctx))
    a = runs[0][0]
    for b, _ in runs[1:]:
        for x, y in zip(a.codes + a.meta + [a.k16, a.v16], b.codes + b.meta + [b.k16, b.v16]):
            assert torch.equal(x, y)
        assert torch.equal(a.v_scale_max[:16], b.v_scale_max[:16])
        for x, y in zip(a.cls_off + a.cls_len + [a.len16], b.cls_off + b.cls_len + [b.len16]):
            n = min(x.numel(), y.numel())
            assert torch.equal(x[:n], y[:n])
    assert (a.v_scale_max[:16] > 0).sum() >= 10


@pytest.mark.parametrize("blocks", [37, 38, 41, 100, 255, 256, 257])
def test_quantizing_a_small_call_on_several_counters(blocks):
    """4 KV heads: 148 and 152 workgroups (one counter, several), odd shares of the counters, 1020, 1024 (the last small call) and 1028;
    the same with an empty 17th sequence (three launches).  Twice on one context: the counters are zero again, also for a decode call."""
    from paper_2605_02262_amd import binding as W
    gen = torch.Generator(device="cuda").manual_seed(blocks)
    heads, hd, group, B = 4, 64, 32, 16
    n = [blocks // B + (1 if b < blocks % B else 0) for b in range(B)]
    seg = [[k // 3, k - k // 3 - k // 4, k // 4, 0] for k in n]
    K, V = (torch.randn(32 * blocks, heads, hd, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    perm = torch.cat([torch.randperm(k, generator=gen, device="cuda") for k in n]).to(torch.int32)
    cap = [32 * sum(s[c] for s in seg) for c in range(3)]
    splits = 4
    ctx = W.Context(W.workspace_bytes(B, 8, hd, splits))
    q = torch.randn(B, 8, hd, generator=gen, device="cuda").to(torch.bfloat16)
    got, out = [], []
    for extra in (1, 0, 0):
        one = [0] * extra
        pk = W.PackedKV(B + extra, heads, hd, group, torch.bfloat16, cap, [0] * (B + 1 + extra), fill=0)
        W.wq_reorder_quantize(ctx, K, V, _table(_offsets([32 * k for k in n] + one)), _table([32] * B + [1] * extra), _table(_offsets(n + one)), perm,
                              _table(seg + [[0] * 4] * extra), 32 * blocks, pk)
        assert ctx.device_status() == 0
        got.append(pk)
        if not extra:
            out.append(W.wq_decode_attention(ctx, q, pk, hd ** -0.5, splits, 32 * max(n), W.DECODE_AUTO | W.DECODE_FIXED_SHARES))
    for b in got[1:]:
        for x, y in zip(got[0].codes + got[0].meta + [got[0].v_scale_max[:B]], b.codes + b.meta + [b.v_scale_max[:B]]):
            assert torch.equal(x, y)
    assert (got[0].v_scale_max[:B] > 0).all() and torch.equal(out[0], out[1]) and torch.isfinite(out[0]).all()


@pytest.mark.parametrize("B", [17, 63, 64, 65, 150])
@pytest.mark.parametrize("short", ["fits", "classes", "rows"])
def test_plan_of_many_sequences(B, short):
    """The tables of a larger call, 64 sequences at a time, against one sequence after the other; with capacities that a sequence in
    the middle and the last ones do not fit (smaller ones behind them still do); the largest value scales against the metadata."""
    from paper_2605_02262_amd import binding as W
    gen = torch.Generator(device="cuda").manual_seed(B)
    heads, hd, group = 2, 64, 32
    win = [(7 * b) % 40 + 1 for b in range(B)]
    seg = [[(b + c) % 3 for c in range(4)] for b in range(B)]
    seg[B // 2] = [9, 9, 9, 0]
    n_win = [sum(s) for s in seg]
    rows = [n * w + b % 4 for b, (n, w) in enumerate(zip(n_win, win))]
    pad = lambda n: (n + 31) // 32 * 32  # noqa: E731
    cap = [sum(pad(s[c] * w) for s, w in zip(seg, win)) for c in range(3)]
    n16 = [s[3] * w + r - n * w for s, w, r, n in zip(seg, win, rows, n_win)]
    room = list(n16)
    if short == "classes":
        cap = [max(32, c - pad(9 * win[B // 2]) - 64) for c in cap]
    if short == "rows":
        room[3] -= 1
        room[-1] = max(0, room[-1] - 1)
    K, V = (torch.randn(sum(rows), heads, hd, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    perm = torch.cat([torch.randperm(n, generator=gen, device="cuda") for n in n_win]).to(torch.int32)
    ctx = W.Context(W.workspace_bytes(B))
    pk = W.PackedKV(B, heads, hd, group, torch.bfloat16, cap, _offsets(room), fill=0)
    W.wq_reorder_quantize(ctx, K, V, _table(_offsets(rows)), _table(win), _table(_offsets(n_win)), perm, _table(seg), sum(rows), pk)
    want, top = 0, [0.0] * B
    for c in range(3):
        off, lens = [0], []
        for s, w in zip(seg, win):
            n = s[c] * w
            if off[-1] + pad(n) > cap[c]:
                n, want = 0, want | W.DEV_CLASS_OVERFLOW
            lens.append(n)
            off.append(off[-1] + pad(n))
        assert pk.cls_off[c].tolist() == off and pk.cls_len[c].tolist() == lens, c
        words = pk.meta[c].view(torch.int32).view(2, heads, cap[c] * (hd // group))[1]
        scales = (words & 0xFFFF).to(torch.int16).view(torch.float16).float()
        for b in range(B):
            part = scales[:, off[b] * (hd // group):off[b + 1] * (hd // group)]
            top[b] = max(top[b], float(part.max()) if part.numel() else 0.0)
    fits = [r >= n for r, n in zip(room, n16)]
    if not all(fits):
        want |= W.DEV_SEG16_OVERFLOW
    assert pk.len16.tolist() == [n if ok else 0 for n, ok in zip(n16, fits)]
    assert pk.v_scale_max[:B].tolist() == top
    assert ctx.device_status() == want


@pytest.mark.parametrize("sizes", [(1, 2, 3), (63, 64, 65), (16,), (128, 129, 0), (191, 193), (256, 257), (319,)])
def test_widths_counted_by_parts(sizes):
    """Sequences of up to 320 windows, one to five chunks of 64 that 16, 8, 5, 4 and 3 parts of the keys are counted for: bit for
    bit against the oracle, ties, NaN and infinities among the scores."""
    from tests.test_gpu_parity import test_assign_bits_few_and_many_windows as check
    check(sizes)
