"""Tier-map and chunk-index bookkeeping of pack and unpack at its edges (whole
and ragged map words, batches held in registers and past them, grouped rows at
odd addresses) against the oracle, byte for byte."""
import pytest

from gpu_helpers import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu

# 16 tokens per map word, 256 per chunk, 131072 per batch of words, 262144 held
LENGTHS = [8, 15, 16, 17, 31, 255, 257, 4113, 131071, 131073, 262144, 262161, 400001]


def shuffled(cfg, n, seed):
    p = skv.plan_tiers(cfg)
    s = p["n_sink"]
    tier = np.repeat(np.array([0, 1, 2, 3], np.uint8), [p["n_fp16"], p["n_int8"], p["n_int4"], p["n_drop"]])
    np.random.default_rng(seed).shuffle(tier)
    return np.concatenate([np.zeros(s, np.uint8), tier])


@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("b,tiers,q4", [(0.45, 3, 0), (0.2, 3, 0), (0.3, 2, 0), (0.4, 3, skv.QUANT_ASYM | skv.QUANT_FP16)])
def test_map_and_index(n, b, tiers, q4):
    say(f"map n={n} b={b} tiers={tiers} q4={q4}")
    cfg, ocfg = configs(1, 1, 32, n, b, tiers, rho=0.01, decay=0.0005, q4=q4)
    k, v = workloads.make_kv(1, 1, n, 32, seed=n)
    tier = shuffled(cfg, n, n)
    want = oracle.pack(ocfg, u16(k), u16(v), tier)
    kd, vd = k.cuda(), v.cuda()
    payload = torch.empty(want.size, dtype=torch.uint8, device="cuda")
    status = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    skv.pack(cfg, kd, vd, torch.from_numpy(tier).cuda(), payload, status)
    assert status.item() == 0
    assert np.array_equal(payload.cpu().numpy(), want)
    nb = workloads.blocks_for(n)
    bt = workloads.make_block_table(n, 16, nb, seed=n)
    kc, vc, st = gpu_decode(cfg, payload, 1, 1, 32, n, 16, nb, bt.cuda())
    okc, ovc, _ = oracle_decode(ocfg, want, 1, 1, 32, 16, nb, bt.numpy())
    assert st == 0 and np.array_equal(u16(kc), okc) and np.array_equal(u16(vc), ovc)
    # a code past the last tier, or a count off by one, in the last token
    for code in (4, 255, (int(tier[-1]) + 1) % 4):
        bad = tier.copy()
        bad[-1] = code
        marked = torch.full_like(payload, 0x5A)
        skv.pack(cfg, kd, vd, torch.from_numpy(bad).cuda(), marked, status)
        assert status.item() == skv.ERR_INVALID_ARG
        assert int(marked[148:152].view(torch.int32).item()) == skv.ERR_INVALID_ARG
        assert bool((marked[256:] == 0x5A).all()), "only the header is written"
    # a map, index or block-table entry that does not fit, at either end
    last_word = 256 + 4 * ((n - 1) // 16)
    cidx = 256 + -(-((n + 3) // 4) // 256) * 256
    for at, bit in ((256, 1), (last_word + ((n - 1) % 16) // 4, 1 << (2 * ((n - 1) % 4))), (cidx, 1)):
        p2 = payload.clone()
        p2[at] ^= bit
        _, _, st = gpu_decode(cfg, p2, 1, 1, 32, n, 16, nb, bt.cuda())
        assert st == skv.ERR_FORMAT, at
    wrong = bt.clone()
    wrong[-1] = nb
    _, _, st = gpu_decode(cfg, payload, 1, 1, 32, n, 16, nb, wrong.cuda())
    assert st == skv.ERR_FORMAT


@pytest.mark.parametrize("n", [9, 17, 1031, 4111])
def test_grouped_rows_at_odd_addresses(n):
    L, H, d = 3, 2, 32
    say(f"grouped map n={n}")
    cfg, ocfg = configs(L, H, d, n, 0.45, rho=0.01)
    gr = skv.Groups(skv.GROUP_HEAD)
    tier = np.stack([shuffled(cfg, n, g) for g in range(L * H)])
    k, v = workloads.make_kv(L, H, n, d, seed=n)
    want = oracle.pack_groups(ocfg, 2, u16(k), u16(v), tier)
    ws = torch.empty(skv.group_workspace_size(cfg, gr), dtype=torch.uint8, device="cuda")
    skv.prepare_groups(cfg, gr, ws)
    payload = torch.empty(skv.grouped_payload_size(cfg, gr), dtype=torch.uint8, device="cuda")
    status = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    skv.pack_groups(cfg, gr, k.cuda(), v.cuda(), torch.from_numpy(tier).cuda(), ws, payload, status)
    assert status.item() == 0 and np.array_equal(payload.cpu().numpy(), want)
    bad = tier.copy()
    bad[-1, -1] = 6
    skv.pack_groups(cfg, gr, k.cuda(), v.cuda(), torch.from_numpy(bad).cuda(), ws, payload, status)
    assert status.item() == skv.ERR_INVALID_ARG
