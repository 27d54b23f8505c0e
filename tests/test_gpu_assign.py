"""The one-workgroup tier cut at its edges against the oracle, exactly: row
lengths around its two instances, and score distributions that leave a cut's
first bin nearly empty, just full and overfull, down to the last digit."""
import pytest

from gpu_helpers import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 3, 63, 65, 257, 1024, 1025, 4097, 8192, 8193, 8200, 20001, 32768, 33000]
KINDS = ["decay", "normal", "constant", "two", "zeros", "outliers", "close", "bad", "near"]


def scores_of(kind, n, rng):
    if kind == "decay":
        return rng.random(n) * np.exp(-0.01 * np.arange(n)[::-1])
    if kind == "normal":
        return rng.normal(size=n)  # half of them rank as +0
    if kind == "constant":
        return np.full(n, 3.25)
    if kind == "two":
        return np.where(rng.random(n) < 0.5, 1.0, 1.0 + 2.0**-30)
    if kind == "zeros":
        return np.where(rng.random(n) < 0.9, 0.0, rng.random(n))
    if kind == "outliers":  # the keys' range is far wider than where most keys lie
        s = 1.0 + rng.random(n) * 1e-6
        s[rng.integers(0, n)] = 1e300
        s[rng.integers(0, n)] = 5e-324
        return s
    if kind == "close":  # equal in the high word, different below it
        return 1.0 + rng.integers(0, 2**11, n) * 2.0**-32
    if kind == "near":  # equal to the last fraction bit that ranks: the token decides
        return 1.0 + rng.integers(0, 3, n) * 2.0**-33
    s = rng.random(n)
    s[rng.random(n) < 0.2] = np.nan
    s[rng.random(n) < 0.1] = np.inf
    s[rng.random(n) < 0.1] = -1.0
    return s


@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("kind", KINDS)
def test_cut_is_the_oracles(n, kind):
    rng = np.random.default_rng(n)
    for b, tiers, rho in ((0.5, 3, 0.01), (0.7, 3, 0.01), (0.2, 3, 0.0), (0.3, 2, 0.02), (1.0, 3, 0.0), (0.26, 3, 0.0)):
        cfg, ocfg = configs(1, 1, 32, n, b, tiers, rho=rho, decay=0.0005)
        try:
            oracle.plan(ocfg)
        except oracle.OracleError:
            continue
        say(f"assign n={n} {kind} b={b} tiers={tiers}")
        s = scores_of(kind, n, rng)
        want = oracle.assign(ocfg, s)
        tier = torch.full((n,), 77, dtype=torch.uint8, device="cuda")
        skv.assign_tiers(cfg, torch.from_numpy(s).cuda(), tier)
        assert np.array_equal(tier.cpu().numpy(), want)


@pytest.mark.parametrize("n,m", [(2047, 2000), (2049, 2000), (65536, 32768), (65537, 32768), (140000, 32768), (600000, 30000),
                                 (2**21, 32768)])
@pytest.mark.parametrize("kind", ["constant", "two", "near"])
def test_ties_are_cut_by_the_token_whatever_its_bits(n, m, kind):
    """Rows of m non-sink tokens behind n - m sinks: the tokens' numbers have up
    to 21 bits, and tied scores leave whole bins to be cut by them."""
    rng = np.random.default_rng(n)
    share = m / n
    for b in (1.0 - 0.55 * share, 1.0 - 0.3 * share):
        cfg, ocfg = configs(1, 1, 32, n, b, 3, num_sink=n - m, decay=0.00001)
        p = oracle.plan(ocfg)
        say(f"assign n={n} m={m} {kind} plan={p}")
        s = scores_of(kind, n, rng)
        tier = torch.full((n,), 77, dtype=torch.uint8, device="cuda")
        skv.assign_tiers(cfg, torch.from_numpy(s).cuda(), tier)
        assert np.array_equal(tier.cpu().numpy(), oracle.assign(ocfg, s))


@pytest.mark.parametrize("ns", [(5, 700, 8192, 1), (8193, 12, 30000), (40000, 100, 9000)])
def test_batched_rows_of_both_instances(ns):
    rng = np.random.default_rng(sum(ns))
    rows = [scores_of("decay", n, rng) for n in ns]
    cfg, ocfg = configs(1, 1, 32, max(ns), 0.6, rho=0.0, decay=0.0005)
    tiers = [torch.full((n,), 77, dtype=torch.uint8, device="cuda") for n in ns]
    skv.assign_batch(cfg, [torch.from_numpy(s).cuda() for s in rows], tiers)
    for n, s, t in zip(ns, rows, tiers):
        _, oc = configs(1, 1, 32, n, 0.6, rho=0.0, decay=0.0005)
        assert np.array_equal(t.cpu().numpy(), oracle.assign(oc, s)), n


@pytest.mark.parametrize("n", [7, 4097, 9001])
def test_grouped_rows_at_odd_addresses(n):
    rng = np.random.default_rng(n)
    L, H = 3, 2
    cfg, ocfg = configs(L, H, 32, n, 0.45, rho=0.01, decay=0.0005)
    gr = skv.Groups(skv.GROUP_HEAD)
    s = np.stack([scores_of(KINDS[g % len(KINDS)], n, rng) for g in range(L * H)])
    ws = torch.empty(skv.group_workspace_size(cfg, gr), dtype=torch.uint8, device="cuda")
    skv.prepare_groups(cfg, gr, ws)
    tier = torch.full((L * H, n), 77, dtype=torch.uint8, device="cuda")
    skv.assign_groups(cfg, gr, torch.from_numpy(s).cuda(), tier, ws)
    assert np.array_equal(tier.cpu().numpy(), oracle.assign_groups(ocfg, 2, s))
