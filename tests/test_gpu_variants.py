"""Quantizer-variant row kernels where their launches change form (short and
long launches, key chunks on their own, per-channel tiers with and without rows
and with non-finite channels), against the oracle byte for byte."""
import pytest

from gpu_helpers import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu

C, A, F = skv.QUANT_CHANNEL, skv.QUANT_ASYM, skv.QUANT_FP16
PAIRS = [(F, A | F), (C | A | F, C | A | F), (C, C), (C | F, A), (A | skv.QUANT_GROUP64, C | A)]


@pytest.mark.parametrize("d", [32, 64, 128, 256])
@pytest.mark.parametrize("q8,q4", PAIRS)
@pytest.mark.parametrize("shape", [(48, 65, 3), (2, 3, 515)], ids=["long", "short"])
@pytest.mark.parametrize("special", [False, True], ids=["plain", "special"])
def test_variant_launches(d, q8, q4, shape, special):
    L, H, n = shape
    say(f"variant d={d} q8={q8} q4={q4} {shape} special={special}")
    cfg, ocfg = configs(L, H, d, n, 0.45 if n > 3 else 0.5, rho=0.01 if n > 3 else 0.0, q8=q8, q4=q4)
    k, v = workloads.make_kv(L, H, n, d, seed=n + d)
    if special:
        k, v = plant_specials(k, v, seed=d)
    otier = oracle.assign(ocfg, np.random.default_rng(d).random(n))
    want = oracle.pack(ocfg, u16(k), u16(v), otier)
    payload = torch.full((want.size,), 0x5A, dtype=torch.uint8, device="cuda")
    status = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    skv.pack(cfg, k.cuda(), v.cuda(), torch.from_numpy(otier).cuda(), payload, status)
    assert status.item() == 0
    diff = np.nonzero(payload.cpu().numpy() != want)[0]
    assert diff.size == 0, diff[:8]
    bs = 4
    nb = workloads.blocks_for(n, bs)
    bt = workloads.make_block_table(n, bs, nb, seed=d)
    kc, vc, st = gpu_decode(cfg, payload, L, H, d, n, bs, nb, bt.cuda())
    okc, ovc, _ = oracle_decode(ocfg, want, L, H, d, bs, nb, bt.numpy())
    assert st == 0 and np.array_equal(u16(kc), okc) and np.array_equal(u16(vc), ovc)


@pytest.mark.parametrize("n", [16384, 16385], ids=["parts", "whole"])  # 64 chunks a segment, and 65
@pytest.mark.parametrize("q", [C, C | A | F], ids=["sym", "asym"])
def test_long_key_segments(n, q):
    """One launch over eight layers decodes what a launch per layer (few chunks: in parts) does."""
    L, H, d, bs = 8, 4, 256, 16
    say(f"long key segments n={n} q={q}")
    cfg, _ = configs(L, H, d, n, 0.45, rho=0.01, q8=q, q4=q)
    gen = torch.Generator(device="cuda").manual_seed(n + q)
    k, v = (torch.randn(L, H, n, d, generator=gen, device="cuda", dtype=torch.float16) for _ in range(2))
    codec = gpu_encode(cfg, k, v)
    nb = workloads.blocks_for(n, bs)
    bt = workloads.make_block_table(n, bs, nb, seed=n).cuda()
    kc, vc, st = gpu_decode(cfg, codec.payload, L, H, d, n, bs, nb, bt)
    ko, vo = caches(L, nb, bs, H, d, "cuda")
    status = [torch.full((1,), -1, dtype=torch.int32, device="cuda")]
    for l in range(L):
        skv.unpack_batch(cfg, [codec.payload], [n], [bt], ko, vo, bs, status, layer_begin=l, layer_count=1)
    assert st == 0 and status[0].item() == 0
    assert torch.equal(kc.view(torch.int16), ko.view(torch.int16))
    assert torch.equal(vc.view(torch.int16), vo.view(torch.int16))
