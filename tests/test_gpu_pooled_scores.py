"""Pooled scoring in three and four launches: the text's pieces in flight, and how a window finds its sequence, at their edges."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n_txt,dim,times", [
    ([1, 300], 8, 1),                       # one lane has a piece
    ([31, 300], 512, 1),                    # a piece per lane; less than one round of the 32 token slices
    ([32, 33, 255, 256], 520, 1),
    ([257, 0, 511, 513], 4096, 1),          # eight pieces per lane; a round more than eight of the slices; no text
    ([600], 4104, 1),                       # ... and one piece more
    ([9] * 63 + [200], 64, 1),              # a lane per sequence
    ([9] * 63 + [200], 64, 12),           # more rows than the means are made with: a launch of their own
    ([5] * 64 + [200], 64, 12),
    ([5] * 64 + [200], 64, 1),              # more sequences than lanes
])
def test_pooled_scores(n_txt, dim, times, dtype):
    """Windows of 7 rows and of 130 (more than two per lane) in turn, rows at the end that fill none, sequences without rows.  float64 reference; fp32 sums of a
    few thousand terms: 1e-5 of the scores' size, 1 / sqrt(dim), is far above their rounding."""
    from paper_2605_02262_amd import binding as W
    gen = torch.Generator(device="cuda").manual_seed(dim + len(n_txt))
    size = [7 if b % 2 else 130 for b in range(len(n_txt))]
    n_win = [0 if b % 5 == 4 else (3 + b % 3) * times for b in range(len(n_txt))]
    n_vis = [w * s + b % 4 for b, (w, s) in enumerate(zip(n_win, size))]
    vis = torch.randn(sum(n_vis), dim, generator=gen, device="cuda").add_(0.2).to(dtype)
    txt = torch.randn(sum(n_txt), dim, generator=gen, device="cuda").add_(0.2).to(dtype)
    table = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")  # noqa: E731
    starts = lambda v: table([sum(v[:i]) for i in range(len(v) + 1)])  # noqa: E731
    ctx = W.Context(W.workspace_bytes(len(n_txt), 0, 0, 0, sum(n_vis), sum(n_txt), dim))
    got = W.wq_window_scores(ctx, vis, txt, starts(n_vis), starts(n_txt), table(size), starts(n_win), sum(n_vis), sum(n_txt), sum(n_win))
    want, v0, t0 = [], 0, 0
    for m, n, w, s in zip(n_vis, n_txt, n_win, size):
        v, t = vis[v0:v0 + w * s].double(), txt[t0:t0 + n].double()
        unit = (t / t.norm(dim=1, keepdim=True)).mean(0) if n else torch.zeros(dim, dtype=torch.float64, device="cuda")
        want.append(((v @ unit) / v.norm(dim=1)).view(w, s).mean(1))
        v0, t0 = v0 + m, t0 + n
    assert times == 1 or sum(n_vis) > 1 << 17
    assert (got.double() - torch.cat(want)).abs().max().item() <= 1e-5 / dim ** 0.5


@pytest.mark.parametrize("front,size,first", [(64, 16, 0), (63, 7, 0), (21, 7, 0), (5, 7, 0), (390, 130, 0), (64, 16, 4), (40, 7, 5)])
def test_rows_in_front_of_the_first_sequence(front, size, first):
    """vis_off[0] = front, whole numbers of windows and not; windows counted from 0 or from `first` (then the rows in front hold the ones before it).
    Twice on one context, whose workspace the first call leaves as it is, and with more rows than the means are made with: the same bits, nothing
    written in front of the scores or behind them; float64 reference, bound as above."""
    from paper_2605_02262_amd import binding as W
    gen = torch.Generator(device="cuda").manual_seed(front + size)
    dim, n_txt, sizes, n_win, guard = 64, [300, 20], [size, 11], [10, 6], 128
    rows = [10 * size + 3, 6 * 11 + 1]
    vis = torch.randn(front + sum(rows) + (1 << 17), dim, generator=gen, device="cuda").add_(0.2).to(torch.bfloat16)
    txt = torch.randn(sum(n_txt), dim, generator=gen, device="cuda").add_(0.2).to(torch.bfloat16)
    table = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")  # noqa: E731
    win_off, total_win = [first, first + 10, first + 16], first + 16
    got, ctx = [], None
    for more in (0, 0, 1 << 17):
        vis_off = [front, front + rows[0], front + sum(rows) + more]
        if more or ctx is None:
            ctx = W.Context(W.workspace_bytes(2, 0, 0, 0, vis_off[-1], sum(n_txt), dim))
        out = torch.full((guard + total_win + guard,), 7.0, device="cuda")
        W.wq_window_scores(ctx, vis[:vis_off[-1]], txt, table(vis_off), table([0, 300, 320]), table(sizes), table(win_off), vis_off[-1], sum(n_txt), total_win,
                           scores=out[guard:guard + total_win])
        assert (out[:guard] == 7.0).all() and (out[guard + total_win:] == 7.0).all()
        got.append(out[guard:guard + total_win])
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    want, n0 = [], 0
    for b, t in enumerate(n_txt):
        unit = torch.nn.functional.normalize(txt[n0:n0 + t].double(), dim=1).mean(0)
        lo, n = (front - first * size, first + 10) if b == 0 else (front + rows[0], 6)
        v = vis[lo:lo + n * sizes[b]].double()
        want.append(((v @ unit) / v.norm(dim=1)).view(n, sizes[b]).mean(1))
        n0 += t
    assert (got[0].double() - torch.cat(want)).abs().max().item() <= 1e-5 / dim ** 0.5


@pytest.mark.parametrize("dim,size", [(1024, 3), (4096, 1)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_as_many_windows_as_there_is_room_to_count(dim, size, dtype):
    """A text of 4 tokens leaves room for the counters of dim / 2 windows (cleared 256 at a time): that many, one more (four launches) and fewer, on one
    context whose workspace holds other bytes: the same bits.  float64 reference, bound as above."""
    from paper_2605_02262_amd import binding as W
    gen = torch.Generator(device="cuda").manual_seed(dim)
    most = dim // 2
    vis = torch.randn((most + 1) * size, dim, generator=gen, device="cuda").add_(0.2).to(dtype)
    txt = torch.randn(4, dim, generator=gen, device="cuda").add_(0.2).to(dtype)
    table = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")  # noqa: E731
    ctx = W.Context(W.workspace_bytes(1, 0, 0, 0, (most + 1) * size, 4, dim))
    got = []
    for n in (most, most + 1, 300):
        ctx.ws[16384:] = 0x5A
        got.append(W.wq_window_scores(ctx, vis[:n * size], txt, table([0, n * size]), table([0, 4]), table([size]), table([0, n]), n * size, 4, n))
    assert torch.equal(got[0], got[1][:most]) and torch.equal(got[2], got[1][:300])
    unit, v = torch.nn.functional.normalize(txt.double(), dim=1).mean(0), vis.double()
    want = ((v @ unit) / v.norm(dim=1)).view(-1, size).mean(1)
    assert (got[1].double() - want).abs().max().item() <= 1e-5 / dim ** 0.5


@pytest.mark.parametrize("n_txt,dim", [([1, 300], 2040), ([127, 128, 129], 2048), ([300], 2056), ([97, 160, 161, 31], 1536)])
def test_pieces_in_flight(n_txt, dim):
    """Four pieces of a row per lane, one more and one less than they hold; four rounds of the 32 token slices and beside it."""
    test_pooled_scores(n_txt, dim, 1, torch.bfloat16)


def test_one_context_for_calls_of_other_shapes():
    """Windows' counters lie behind what depends on a call's sizes: calls of several shapes in turn on one context, twice, have the bits that each has on
    one of its own."""
    from paper_2605_02262_amd import binding as W
    gen = torch.Generator(device="cuda").manual_seed(7)
    table = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")  # noqa: E731
    starts = lambda v: table([sum(v[:i]) for i in range(len(v) + 1)])  # noqa: E731
    calls = []
    for n_txt, n_win, size, dim in (([300], [40], 33, 512), ([20, 400], [3, 500], 7, 256), ([260], [1], 1500, 128), ([5] * 70, [9] * 70, 5, 1024), ([299], [41], 33, 512)):
        rows = [n * size + b % 3 for b, n in enumerate(n_win)]
        vis = torch.randn(sum(rows), dim, generator=gen, device="cuda").to(torch.bfloat16)
        txt = torch.randn(sum(n_txt), dim, generator=gen, device="cuda").to(torch.bfloat16)
        calls.append((vis, txt, starts(rows), starts(n_txt), table([size] * len(rows)), starts(n_win), sum(rows), sum(n_txt), sum(n_win)))
    need = [W.workspace_bytes(c[4].numel(), 0, 0, 0, c[6], c[7], c[0].shape[1]) for c in calls]
    own = [W.wq_window_scores(W.Context(n), *c) for n, c in zip(need, calls)]
    ctx = W.Context(max(need))
    for _ in range(2):
        for c, want in zip(calls, own):
            assert torch.equal(W.wq_window_scores(ctx, *c), want) and torch.isfinite(want).all()
