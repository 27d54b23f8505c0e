"""Upgrade row kernels at the edges of their workgroups: 4 rows per thread, so
256 / 128 / 64 / 32 listed rows per workgroup at d = 32 / 64 / 128 / 256, every
tier next to every other in a wave, and more (layer, head) pairs than one grid
dimension holds.  Bytes and caches must equal the oracle's."""
import pytest

from gpu_helpers import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu


def _check(L, H, d, n, m, mode, specials):
    say(f"upgrade rows L={L} H={H} d={d} n={n} m={m} mode={mode}")
    cfg, ocfg = configs(L, H, d, n, 0.5, 3)
    rng = np.random.default_rng(d + m)
    k, v = workloads.make_kv(L, H, n, d, seed=m)
    if specials:
        plant_specials(k, v, m)
    tier = rng.integers(0, 4, size=n).astype(np.uint8)
    tokens = np.sort(rng.choice(n, size=m, replace=False)).astype(np.int32)
    want = oracle.pack_upgrade(ocfg, u16(k), u16(v), tier, tokens, mode)
    up = torch.full((want.size,), 0xA5, dtype=torch.uint8, device="cuda")
    st = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    skv.pack_upgrade(cfg, k.cuda(), v.cuda(), torch.from_numpy(tier).cuda(), torch.from_numpy(tokens).cuda(), mode, up,
                     st)
    assert int(st.item()) == 0
    bad = np.flatnonzero(up.cpu().numpy() != want)
    assert bad.size == 0, f"{bad.size} bytes differ, first at {bad[:8]}"

    bs = 5
    nb = -(-n // bs) + 2
    table = rng.permutation(nb)[: -(-n // bs)].astype(np.int32)
    caches = [rng.standard_normal((L, nb, bs, H, d)).astype(np.float16).view(np.uint16) for _ in range(2)]
    kc, vc = (torch.from_numpy(c.view(np.float16).copy()).cuda() for c in caches)
    skv.unpack_upgrade(cfg, up, m, mode, kc, vc, torch.from_numpy(table).cuda(), bs, st)
    assert int(st.item()) == 0
    assert oracle.unpack_upgrade(ocfg, want, *caches, table, bs) == 0
    assert np.array_equal(u16(kc.cpu()), caches[0]) and np.array_equal(u16(vc.cpu()), caches[1])


@pytest.mark.parametrize("mode", (skv.UPGRADE_FP16, skv.UPGRADE_RESIDUAL8))
@pytest.mark.parametrize("d", (32, 64, 128, 256))
@pytest.mark.parametrize("extra", (-1, 0, 1))
def test_workgroup_edges(mode, d, extra):
    _check(2, 3, d, 700, 8192 // d + extra, mode, specials=True)


@pytest.mark.parametrize("mode", (skv.UPGRADE_FP16, skv.UPGRADE_RESIDUAL8))
def test_more_pairs_than_a_grid_dimension(mode):
    _check(257, 128, 32, 7, 5, mode, specials=False)


@pytest.mark.parametrize("mode", (skv.UPGRADE_FP16, skv.UPGRADE_RESIDUAL8))
@pytest.mark.parametrize("d", (32, 64, 128, 256))
@pytest.mark.parametrize("groups", (2, 3, 8, 9))
def test_lists_of_few_workgroups(mode, d, groups):
    """The workgroups of a pair begin at a scattered one up to 4 (d = 32) or 16 of
    them (twice `groups`: K and V), at the first beyond; the last holds one row."""
    m = (groups - 1) * (8192 // d) + 1
    _check(3, 5, d, m + 9, m, mode, specials=False)
