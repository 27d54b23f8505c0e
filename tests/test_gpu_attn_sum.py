"""The sum of an attention score over the (layer, KV head) pairs: skv_score,
skv_score_static and skv_score_groups with one group agree bit for bit.

A per-head grouped score with decay 0 and a power of two of observation rows is
the pair's binary32 column sum, scaled exactly, so the sum is also checked
against those.  The queries are scaled so that one token's column sums span far
more than the 29 bits by which binary64 exceeds binary32: another order of
addition shows in the last bits."""
import pytest

from gpu_helpers import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu

# (L, H, d, n): a single pair, fewer pairs than parts of the sum, numbers of
# pairs that do not split evenly, several batches of loads per part
SHAPES = [(1, 1, 64, 70), (2, 3, 256, 1), (3, 7, 64, 333), (5, 13, 128, 300), (43, 3, 32, 64), (67, 5, 32, 191)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_every_entry_point_adds_alike(shape):
    L, H, d, n = shape
    say(f"attention sum {shape}")
    Hq, W = 2 * H, 8
    cfg, _ = configs(L, H, d, n, 1.0, decay=0.0, rho=0.0, mode=oracle.ATTN, Hq=Hq, W=W)
    k, v = workloads.make_kv(L, H, n, d, seed=n, device="cuda")
    q = (workloads.make_qobs(L, Hq, W, d, seed=n, device="cuda") * 6).contiguous()

    def grouped(gran):
        gr = skv.Groups(gran)
        ws = torch.empty(skv.group_workspace_size(cfg, gr), dtype=torch.uint8, device="cuda")
        skv.prepare_groups(cfg, gr, ws)
        out = torch.empty(skv.group_count(cfg, gr), n, dtype=torch.float64, device="cuda")
        skv.score_groups(cfg, gr, k, v, q, out, ws)
        return out.cpu().numpy()

    ws = torch.empty(skv.workspace_size(cfg), dtype=torch.uint8, device="cuda")
    skv.prepare(cfg, ws)
    score, static = (torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2))
    skv.score(cfg, k, v, q, score, ws)
    skv.score_static(cfg, k, v, q, static)
    score = score.cpu().numpy()
    assert np.array_equal(bits64(static.cpu().numpy()), bits64(score))
    assert np.array_equal(bits64(grouped(skv.GROUP_TOKEN)[0]), bits64(score))
    if L == 1:
        assert np.array_equal(bits64(grouped(skv.GROUP_LAYER)[0]), bits64(score))

    colsum = grouped(skv.GROUP_HEAD) * 16.0  # 2 query heads x 8 queries per pair
    assert np.array_equal(colsum.astype(np.float32).astype(np.float64), colsum)
    up, down = (np.add.accumulate(c, axis=0)[-1] for c in (colsum, colsum[::-1]))
    if L * H > 8 and n > 1:
        assert not np.array_equal(up, down), "the inputs do not tell orders apart"
    # LH - 1 additions of non-negative values, the product and numpy's own chain
    want = up * (1.0 / (L * Hq * W))
    assert np.all(np.abs(score - want) <= 2 * (L * H + 1) * 2.0**-53 * want)
