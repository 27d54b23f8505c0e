"""Row kernels where their launches change form (workgroups per chunk, runs per
XCD and their incomplete last round, long and short unpack launches), against
the oracle byte for byte."""
import pytest

from gpu_helpers import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu

SHAPES = [  # L, H, d, n, block size
    (1, 1, 32, 524288 + 300, 7),   # one workgroup per chunk, past 4096 workgroups
    (1, 3, 64, 87000, 48),         # two per chunk (pack), ragged last round
    (8, 8, 128, 2000, 16),         # short segments, exactly 4096 workgroups
    (7, 9, 128, 2300, 5),          # short segments, incomplete last round
    (1, 1, 128, 131072 + 77, 16),  # long segments
    (3, 5, 256, 4097, 32),         # eight per chunk (pack), short unpack launch
    (48, 65, 256, 33, 3),          # more than 6144 chunks: the long unpack form
    (2, 2, 256, 1, 16),
]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_pack_and_unpack(shape):
    L, H, d, n, bs = shape
    say(f"rows {shape}")
    cfg, ocfg = configs(L, H, d, n, 1.0 if n == 1 else 0.4, decay=0.0004, rho=0.02 if n > 1 else 0.0)
    k, v = workloads.make_kv(L, H, n, d, seed=n)
    otier = oracle.assign(ocfg, np.random.default_rng(n).random(n))
    want = oracle.pack(ocfg, u16(k), u16(v), otier)
    payload = torch.full((want.size,), 0x5A, dtype=torch.uint8, device="cuda")
    status = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    skv.pack(cfg, k.cuda(), v.cuda(), torch.from_numpy(otier).cuda(), payload, status)
    assert status.item() == 0 and np.array_equal(payload.cpu().numpy(), want)
    nb = workloads.blocks_for(n, bs) + 2
    bt = workloads.make_block_table(n, bs, nb, seed=n)
    kc, vc, st = gpu_decode(cfg, payload, L, H, d, n, bs, nb, bt.cuda())
    okc, ovc, _ = oracle_decode(ocfg, want, L, H, d, bs, nb, bt.numpy())
    assert st == 0 and np.array_equal(u16(kc), okc) and np.array_equal(u16(vc), ovc)


def test_batch_split_over_launches():
    """Requests whose chunks together pass a launch's limit take several: they share their K/V here."""
    L, H, d, n = 64, 513, 32, 3
    cfg, ocfg = configs(L, H, d, n, 0.5, rho=0.0)
    k, v = workloads.make_kv(L, H, n, d, seed=1)
    kd, vd = k.cuda(), v.cuda()
    count = 17  # 65664 chunks each: 15 fill a launch
    rng = np.random.default_rng(3)
    otiers = [oracle.assign(ocfg, rng.random(n)) for _ in range(count)]
    tiers = [torch.from_numpy(t).cuda() for t in otiers]
    say("batch of 17 x 65664 chunks")
    payloads = [torch.zeros(skv.payload_size(cfg), dtype=torch.uint8, device="cuda") for _ in range(count)]
    skv.pack_batch(cfg, [kd] * count, [vd] * count, tiers, payloads)
    nb = count
    kc, vc = caches(L, nb, 4, H, d, "cuda")
    st = torch.full((count,), 9, dtype=torch.int32, device="cuda")
    tables = [torch.tensor([i], dtype=torch.int32, device="cuda") for i in range(count)]
    skv.unpack_batch(cfg, payloads, [n] * count, tables, kc, vc, 4, [st[i:i + 1] for i in range(count)])
    assert st.cpu().tolist() == [0] * count
    for i in (0, 14, 15, 16):
        want = oracle.pack(ocfg, u16(k), u16(v), otiers[i])
        assert np.array_equal(payloads[i].cpu().numpy(), want), i
        okc, ovc, _ = oracle_decode(ocfg, want, L, H, d, 4, 1, np.zeros(1, np.int32))
        assert np.array_equal(u16(kc[:, i:i + 1].contiguous()), okc) and np.array_equal(u16(vc[:, i:i + 1].contiguous()), ovc)
