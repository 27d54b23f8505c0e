"""Unpack on both sides of its smallest launches (several workgroups per chunk at
head dimensions 64 and 32 up to 512 chunks), one map and grouped, against the
oracle byte for byte."""
import pytest

from gpu_helpers import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu

SHAPES = [  # L, H, d, n, block size
    (1, 1, 64, 1, 16),
    (1, 2, 64, 257, 7),
    (2, 1, 32, 255, 3),
    (4, 8, 64, 2048, 16),  # 512 chunks
    (16, 8, 32, 500, 5),
    (3, 19, 64, 1200, 16),  # 570 chunks
]


@pytest.mark.parametrize("grouped", [False, True], ids=["one_map", "grouped"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_unpack(shape, grouped):
    L, H, d, n, bs = shape
    say(f"tiny unpack {shape} grouped={grouped}")
    cfg, ocfg = configs(L, H, d, n, 1.0 if n == 1 else 0.4, rho=0.0)
    k, v = workloads.make_kv(L, H, n, d, seed=n)
    rng = np.random.default_rng(n)
    nb = workloads.blocks_for(n, bs) + 2
    bt = workloads.make_block_table(n, bs, nb, seed=n)
    if not grouped:
        want = oracle.pack(ocfg, u16(k), u16(v), oracle.assign(ocfg, rng.random(n)))
        kc, vc, st = gpu_decode(cfg, torch.from_numpy(want).cuda(), L, H, d, n, bs, nb, bt.cuda())
        okc, ovc, _ = oracle_decode(ocfg, want, L, H, d, bs, nb, bt.numpy())
        assert st == 0 and np.array_equal(u16(kc), okc) and np.array_equal(u16(vc), ovc)
        return
    gr = skv.Groups(skv.GROUP_HEAD)
    tiers = np.stack([oracle.assign(ocfg, rng.random(n)) for _ in range(L * H)])
    want = oracle.pack_groups(ocfg, 2, u16(k), u16(v), tiers)
    ws = torch.empty(skv.group_workspace_size(cfg, gr), dtype=torch.uint8, device="cuda")
    skv.prepare_groups(cfg, gr, ws)
    kc, vc = caches(L, nb, bs, H, d, "cuda")
    st = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    okc, ovc = u16(kc).copy(), u16(vc).copy()
    skv.unpack_groups(cfg, gr, ws, torch.from_numpy(want).cuda(), kc, vc, bt.cuda(), bs, st)
    assert oracle.unpack_groups(ocfg, 2, want, okc, ovc, bt.numpy(), bs) == 0
    assert st.item() == 0 and np.array_equal(u16(kc), okc) and np.array_equal(u16(vc), ovc)
