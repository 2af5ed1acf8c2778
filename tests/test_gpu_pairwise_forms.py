"""The pairwise scoring kernel's forms (text columns x height of a workgroup's row tiles), each at its edges."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _exact(vis, txt, n_vis, n_txt, window):
    """Mean cosine per window in float64 (by linearity: against the mean unit text vector)."""
    out, v0, t0 = [], 0, 0
    for m, n in zip(n_vis, n_txt):
        v, t = vis[v0:v0 + m].double(), txt[t0:t0 + n].double()
        unit = (t / t.norm(dim=1, keepdim=True)).mean(0) if n else torch.zeros(vis.shape[1], dtype=torch.float64, device=vis.device)
        c = (v @ unit) / v.norm(dim=1)
        out.append(c[:m // window * window].view(-1, window).mean(1))
        v0, t0 = v0 + m, t0 + n
    return torch.cat(out)


@pytest.mark.parametrize("dtype,dim", [(torch.bfloat16, 128), (torch.float16, 384)])
@pytest.mark.parametrize("text", [1, 32, 33, 64, 65, 128, 129, 256, 257])
def test_pairwise_every_form(text, dtype, dim):
    """One sequence beside a short one of another text length; `per` sixteens of rows for each of the 256 workgroups reach every
    tile height (1 to 16 and one more, which takes two tiles), the odd rows at the end a partial tile of 16.  Windows of one row, so
    that every row's score is looked at.  dim 128: fewer steps than the loads are sent ahead; 384: three times as many.  float64
    reference; fp32 sums of a few hundred terms."""
    from paper_2605_02262_amd import binding as W
    gen = torch.Generator(device="cuda").manual_seed(text)
    window = 1
    for per in ([1, 4, 5, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17] if 128 < text <= 256 else [1, 6, 7, 8, 16, 17]):
        n_vis, n_txt = [per * 4096 - 5, 37], [text, 300]
        vis = torch.randn(sum(n_vis), dim, generator=gen, device="cuda").add_(0.05).to(dtype)
        txt = torch.randn(sum(n_txt), dim, generator=gen, device="cuda").add_(0.05).to(dtype)
        table = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")  # noqa: E731
        n_win = [m // window for m in n_vis]
        ctx = W.Context(W.workspace_bytes(2, 0, 0, 0, sum(n_vis), sum(n_txt), dim))
        got = W.wq_window_scores(ctx, vis, txt, table([0, n_vis[0], sum(n_vis)]), table([0, n_txt[0], sum(n_txt)]), table([window, window]),
                                 table([0, n_win[0], sum(n_win)]), sum(n_vis), sum(n_txt), sum(n_win), algo=W.SCORE_PAIRWISE_MFMA)
        want = _exact(vis, txt, n_vis, n_txt, window)
        worst = ((got.double() - want).abs() - 1e-4 * want.abs()).max().item()
        assert worst <= 1e-7, (per, worst)


@pytest.mark.parametrize("n_vis,n_txt", [
    ([4704] * 5, [64] * 5),                                   # 5.7 sixteens of rows a workgroup
    ([3920, 700, 16, 2000], [300, 600, 20, 257]),             # few wide tiles: many workgroups without work
    ([0, 37, 0, 5000, 15], [5, 0, 30, 256, 257]),             # sequences without rows or without text
    ([16] * 64, [3] * 64),                                    # fewer workgroups than the chip has
    ([48] * 65, [40] * 65),                                   # a lane has two sequences
    ([130, 0, 500, 33] * 40 + [7], [200, 3, 20, 300] * 40 + [129]),      # ... three, whole workgroups for each
    ([17, 1000] * 128, [30, 10] * 128),                       # four, too many rows for whole workgroups
    ([37, 96, 5, 97] * 100, [10, 70, 257, 4] * 100),          # more than four: equal shares, sequences of up to 96 rows not cut
    ([4000] + [20] * 600, [150] + [2] * 600),                 # many of them in a share, one sequence over many shares
    ([90000, 1000, 1000, 33000], [10, 200, 10, 10]),          # large shares: equal ones that cross sequences
])
def test_pairwise_whole_workgroups(n_vis, n_txt):
    """Whole numbers of workgroups per sequence where they fit, else equal shares of all rows: every row scored once (windows of one row)."""
    from paper_2605_02262_amd import binding as W
    dim, window = 128, 1
    gen = torch.Generator(device="cuda").manual_seed(len(n_vis))
    vis = torch.randn(sum(n_vis), dim, generator=gen, device="cuda").add_(0.05).bfloat16()
    txt = torch.randn(sum(n_txt), dim, generator=gen, device="cuda").add_(0.05).bfloat16()
    starts = lambda v: torch.tensor([0, *torch.tensor(v).cumsum(0).tolist()], dtype=torch.int32, device="cuda")  # noqa: E731
    n_win = [m // window for m in n_vis]
    ctx = W.Context(W.workspace_bytes(len(n_vis), 0, 0, 0, sum(n_vis), sum(n_txt), dim))
    got = W.wq_window_scores(ctx, vis, txt, starts(n_vis), starts(n_txt), torch.full((len(n_vis),), window, dtype=torch.int32, device="cuda"),
                             starts(n_win), sum(n_vis), sum(n_txt), sum(n_win), algo=W.SCORE_PAIRWISE_MFMA)
    want = _exact(vis, txt, n_vis, n_txt, window)
    assert ((got.double() - want).abs() - 1e-4 * want.abs()).max().item() <= 1e-7
