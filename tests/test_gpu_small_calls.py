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
    for window, n_win, texts in ((16, [3, 0, 2], [16, 3, 0]), (1, [5, 2], [1, 8]), (17, [1, 2], [9, 7]), (64, [1], [33]), (3, [2, 1, 1], [32, 31, 65])):
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
