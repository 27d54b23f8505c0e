"""Tier cuts of long rows that become final before the last digit, exactly:
rows around the edges of the split form's workgroups, cuts that end on
different passes (one on the exponent, one on the last token bits), rows of one
launch that end apart, and the same on one workgroup."""
import pytest

from gpu_helpers import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu

SINKS = 5
LENGTHS = [SINKS + 32769, SINKS + 40960, SINKS + 40961, SINKS + 49151, 100003]


def scores_of(kind, n, rng):
    if kind == "spread":  # final after two or three digits
        return rng.random(n) * np.exp(-0.001 * np.arange(n)[::-1])
    if kind == "constant":  # the token decides: final on the last digits
        return np.full(n, 0.75)
    if kind == "mixed":  # top quarter apart by exponent alone, the rest tied
        return np.where(np.arange(n) % 4 == 1, 4.0, 1.0)
    s = rng.random(n) * np.exp(-0.001 * np.arange(n)[::-1])
    s[rng.random(n) < 0.6] = 0.0  # "zeros": the lowest bin holds most keys
    return s


KINDS = ["spread", "constant", "mixed", "zeros"]


@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("kind", KINDS)
def test_single_row(n, kind):
    s = scores_of(kind, n, np.random.default_rng(n))
    ds = torch.from_numpy(s).cuda()
    for b, tiers in ((0.4, 3), (0.7, 3), (0.15, 3), (0.3, 2), (1.0, 3)):
        say(f"select n={n} {kind} b={b} tiers={tiers}")
        cfg, ocfg = configs(1, 1, 32, n, b, tiers, num_sink=SINKS, decay=1e-3)
        want = oracle.assign(ocfg, s)
        ws = torch.empty(skv.workspace_size(cfg), dtype=torch.uint8, device="cuda")
        for w in (ws, ws, None):  # the scratch is used twice over
            tier = torch.full((n,), 77, dtype=torch.uint8, device="cuda")
            skv.assign_tiers(cfg, ds, tier, ws=w)
            assert np.array_equal(tier.cpu().numpy(), want)


def test_rows_of_one_launch_end_apart():
    n = 41003
    rng = np.random.default_rng(3)
    cfg, ocfg = configs(2, 4, 32, n, 0.45, num_sink=SINKS, decay=1e-3)
    gr = skv.Groups(skv.GROUP_HEAD)
    s = np.stack([scores_of(KINDS[g % 4], n, rng) for g in range(8)])
    ws = torch.empty(skv.group_workspace_size(cfg, gr), dtype=torch.uint8, device="cuda")
    skv.prepare_groups(cfg, gr, ws)
    tier = torch.full((8, n), 77, dtype=torch.uint8, device="cuda")
    skv.assign_groups(cfg, gr, torch.from_numpy(s).cuda(), tier, ws)
    assert np.array_equal(tier.cpu().numpy(), oracle.assign_groups(ocfg, 2, s))
