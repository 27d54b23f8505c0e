"""Requests of one chunk around the edges of its parts (32, 64 or 128 tokens),
whose launches make only the parts that hold tokens, and batches of unlike
lengths, where some parts stay empty: per token, per variant and grouped, against
the oracle byte for byte."""
import pytest

from gpu_helpers import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu

KIVI = skv.QUANT_CHANNEL | skv.QUANT_ASYM | skv.QUANT_FP16


@pytest.mark.parametrize("d", [32, 64, 128, 256])
@pytest.mark.parametrize("shape", [(3, 5), (10, 60)], ids=["few", "many"])  # both sides of 512 chunks
@pytest.mark.parametrize("q", [0, skv.QUANT_FP16, KIVI], ids=["plain", "f16", "kivi"])
def test_one_chunk(d, shape, q):
    L, H = shape
    for n in (1, 31, 32, 33, 64, 65, 128, 129, 192, 193, 255) if shape == (3, 5) else (32, 64, 65, 128, 129, 224, 225):
        say(f"short d={d} {L}x{H} n={n} q={q}")
        cfg, ocfg = configs(L, H, d, n, 1.0 if n == 1 else 0.4, rho=0.0, q8=q, q4=q)
        k, v = workloads.make_kv(L, H, n, d, seed=n)
        otier = oracle.assign(ocfg, np.random.default_rng(n).random(n))
        want = oracle.pack(ocfg, u16(k), u16(v), otier)
        payload = torch.full((want.size,), 0x5A, dtype=torch.uint8, device="cuda")
        skv.pack(cfg, k.cuda(), v.cuda(), torch.from_numpy(otier).cuda(), payload)
        assert np.array_equal(payload.cpu().numpy(), want), n
        bs, nb = 16, workloads.blocks_for(n, 16) + 1
        bt = workloads.make_block_table(n, bs, nb, seed=n)
        kc, vc, st = gpu_decode(cfg, payload, L, H, d, n, bs, nb, bt.cuda())
        okc, ovc, _ = oracle_decode(ocfg, want, L, H, d, bs, nb, bt.numpy())
        assert st == 0 and np.array_equal(u16(kc), okc) and np.array_equal(u16(vc), ovc), n
        if q:
            continue
        gr = skv.Groups(skv.GROUP_LAYER)
        tiers = np.stack([oracle.assign(ocfg, np.random.default_rng(l).random(n)) for l in range(L)])
        want = oracle.pack_groups(ocfg, 1, u16(k), u16(v), tiers)
        ws = torch.empty(skv.group_workspace_size(cfg, gr), dtype=torch.uint8, device="cuda")
        skv.prepare_groups(cfg, gr, ws)
        payload = torch.full((want.size,), 0x5A, dtype=torch.uint8, device="cuda")
        skv.pack_groups(cfg, gr, k.cuda(), v.cuda(), torch.from_numpy(tiers).cuda(), ws, payload)
        assert np.array_equal(payload.cpu().numpy(), want), n
        kc, vc = caches(L, nb, bs, H, d, "cuda")
        okc, ovc = u16(kc).copy(), u16(vc).copy()
        st = torch.full((1,), 9, dtype=torch.int32, device="cuda")
        skv.unpack_groups(cfg, gr, ws, payload, kc, vc, bt.cuda(), bs, st)
        assert oracle.unpack_groups(ocfg, 1, want, okc, ovc, bt.numpy(), bs) == 0
        assert st.item() == 0 and np.array_equal(u16(kc), okc) and np.array_equal(u16(vc), ovc), n


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("ns", [(1, 64, 33, 20), (300, 17, 256, 65, 513)], ids=["one_chunk", "unlike"])
def test_batch(d, ns):
    L, H = 4, 20
    say(f"short batch d={d} {ns}")
    cfg, _ = configs(L, H, d, max(ns), 0.4, rho=0.0)
    reqs, at = [], 0
    for n in ns:
        _, oc = configs(L, H, d, n, 0.4, rho=0.0)
        tier = oracle.assign(oc, np.random.default_rng(n).random(n))
        k, v = workloads.make_kv(L, H, n, d, seed=n)
        nb = workloads.blocks_for(n, 16)
        reqs.append((n, oc, tier, k, v, np.arange(at, at + nb, dtype=np.int32)))
        at += nb
    wants = [oracle.pack(oc, u16(k), u16(v), tier) for _, oc, tier, k, v, _ in reqs]
    payloads = [torch.full((w.size,), 0x5A, dtype=torch.uint8, device="cuda") for w in wants]
    skv.pack_batch(cfg, [r[3].cuda() for r in reqs], [r[4].cuda() for r in reqs],
                   [torch.from_numpy(r[2]).cuda() for r in reqs], payloads)
    for p, w, r in zip(payloads, wants, reqs):
        assert np.array_equal(p.cpu().numpy(), w), r[0]
    kc, vc = caches(L, at, 16, H, d, "cuda")
    okc, ovc = u16(kc).copy(), u16(vc).copy()
    sts = [torch.full((1,), 9, dtype=torch.int32, device="cuda") for _ in reqs]
    skv.unpack_batch(cfg, payloads, list(ns), [torch.from_numpy(r[5]).cuda() for r in reqs], kc, vc, 16, sts)
    assert [s.item() for s in sts] == [0] * len(ns)
    for w, r in zip(wants, reqs):
        assert oracle.unpack(r[1], w, okc, ovc, r[5], 16) == oracle.OK
    assert np.array_equal(u16(kc), okc) and np.array_equal(u16(vc), ovc)
