"""KV-norm scores at the edges of the partial-sum launches, against the oracle
bit for bit (the sums are exact, so no tolerance)."""
import pytest

from gpu_helpers import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu

# (L, H, d, n): one part of 1..4 pairs, several parts of 4 with a rest, parts
# of 8 (more than 4096 workgroups), the largest part (512 pairs) and one past it,
# parts of 2 and just past them (768 workgroups of 4 pairs), and rows of one and
# two pairs on both sides of 4800 workgroups
SHAPES = [(1, 1, 128, 1), (1, 3, 32, 65), (2, 2, 64, 33), (5, 1, 256, 9), (3, 3, 128, 17), (13, 3, 32, 130),
          (1, 33, 32, 70001), (64, 8, 32, 2), (57, 9, 32, 3),
          (3, 3, 64, 8192), (3, 3, 64, 8193), (1, 5, 256, 300), (1, 1, 256, 38400), (1, 1, 256, 38401), (1, 1, 64, 153700),
          (1, 2, 256, 38401), (2, 1, 256, 38400)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("values", ["mixed", "largest", "smallest"])
def test_part_edges_and_extremes(shape, values):
    L, H, d, n = shape
    say(f"score {shape} {values}")
    g = torch.Generator().manual_seed(n)
    if values == "mixed":  # every exponent, inf and NaN among them
        kv = [torch.randint(-32768, 32768, (L, H, n, d), generator=g).to(torch.int16).view(torch.float16) for _ in range(2)]
    else:
        b = 0x7BFF if values == "largest" else 0x0001
        kv = [torch.full((L, H, n, d), b, dtype=torch.int16).view(torch.float16) for _ in range(2)]
    cfg, ocfg = configs(L, H, d, n, 1.0, decay=0.001)
    want = bits64(oracle.score(ocfg, u16(kv[0]), u16(kv[1])))
    k, v = kv[0].cuda(), kv[1].cuda()
    ws = torch.empty(skv.workspace_size(cfg), dtype=torch.uint8, device="cuda")
    skv.prepare(cfg, ws)
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    skv.score(cfg, k, v, None, out, ws)
    assert np.array_equal(bits64(out.cpu().numpy()), want)
    # one map of the whole request
    one = skv.Groups(skv.GROUP_TOKEN)
    ws1 = torch.empty(skv.group_workspace_size(cfg, one), dtype=torch.uint8, device="cuda")
    skv.prepare_groups(cfg, one, ws1)
    o1 = torch.empty(1, n, dtype=torch.float64, device="cuda")
    skv.score_groups(cfg, one, k, v, None, o1, ws1)
    assert np.array_equal(bits64(o1[0].cpu().numpy()), want)
    # batched: one launch shape for both requests, the parts of the whole batch
    outs = [torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2)]
    wsb = torch.empty(skv.batch_workspace_size(cfg, outs), dtype=torch.uint8, device="cuda")
    skv.prepare(cfg, wsb)
    skv.score_batch(cfg, [k, k], [v, v], outs, wsb)
    for o in outs:
        assert np.array_equal(bits64(o.cpu().numpy()), want)
    # per layer: a part that is a whole group writes its score
    ocall = oracle.score_groups(ocfg, 1, u16(kv[0]), u16(kv[1]))
    gr = skv.Groups(skv.GROUP_LAYER)
    wsg = torch.empty(skv.group_workspace_size(cfg, gr), dtype=torch.uint8, device="cuda")
    skv.prepare_groups(cfg, gr, wsg)
    og = torch.empty(L, n, dtype=torch.float64, device="cuda")
    skv.score_groups(cfg, gr, k, v, None, og, wsg)
    assert np.array_equal(bits64(og.cpu().numpy()), bits64(ocall))
