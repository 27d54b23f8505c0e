"""Row launches made in several pieces: requests of very many (layer, head) pairs,
whose flat workgroups pass one launch, against the same request packed and
unpacked layer by layer, byte for byte.  K and V are one buffer, and so are the
two caches (both then receive the same rows)."""
import pytest

from gpu_helpers import *  # noqa: F401,F403

pytestmark = pytest.mark.gpu

L, H = 64, 1023  # 65472 pairs


def _need(nbytes):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < nbytes:
        pytest.skip("not enough free device memory")


def _keys(n, d):
    k = torch.empty(L, H, n, d, dtype=torch.float16, device="cuda")
    flat = k.view(-1)
    some = torch.randn(1 << 25, generator=torch.Generator("cuda").manual_seed(d), device="cuda").half()
    for at in range(0, flat.numel(), some.numel()):
        flat[at:at + some.numel()].copy_(some[:min(some.numel(), flat.numel() - at)])
    return k


def _pack(cfg, k, tier):
    payload = torch.zeros(skv.payload_size(cfg), dtype=torch.uint8, device="cuda")
    st = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    skv.pack(cfg, k, k, tier, payload, st)
    assert st.item() == 0
    return payload


def _equal(a, b):  # outside the assertions, whose messages would print the tensors
    return bool(torch.equal(a.view(torch.uint8), b.view(torch.uint8)))


def _u64(payload, word):
    return int(payload[4 * word:4 * word + 8].view(torch.int64).item())


def test_pack_in_pieces():
    d, n = 256, 4097  # 17 chunks of eight workgroups per segment: more than 2^32 threads
    _need(170 << 30)
    say("pack in pieces")
    cfg, ocfg = configs(L, H, d, n, 0.02, rho=0.0)
    tier = torch.from_numpy(oracle.assign(ocfg, np.random.default_rng(1).random(n))).cuda()
    k = _keys(n, d)
    payload = _pack(cfg, k, tier)
    want = torch.zeros_like(payload)
    for l in range(L):
        skv.pack_batch(cfg, [k], [k], [tier], [want], layer_begin=l, layer_count=1)
    assert _equal(payload, want)
    # one group holds the same rows and scales at its own offset
    gr = skv.Groups(skv.GROUP_TOKEN)
    ws = torch.empty(skv.group_workspace_size(cfg, gr), dtype=torch.uint8, device="cuda")
    skv.prepare_groups(cfg, gr, ws)
    want.zero_()
    grouped = torch.zeros(skv.grouped_payload_size(cfg, gr), dtype=torch.uint8, device="cuda")
    st = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    skv.pack_groups(cfg, gr, k, k, tier, ws, grouped, st)
    assert st.item() == 0
    assert _equal(payload[_u64(payload, 24):], grouped[_u64(grouped, 28):])


def test_unpack_in_pieces():
    d, n, bs = 128, 2049, 16  # 9 chunks of four workgroups per segment: more than 2^30 threads
    _need(120 << 30)
    say("unpack in pieces")
    cfg, ocfg = configs(L, H, d, n, 0.1, rho=0.0)
    tier = torch.from_numpy(oracle.assign(ocfg, np.random.default_rng(2).random(n))).cuda()
    payload = _pack(cfg, _keys(n, d), tier)
    nb = workloads.blocks_for(n, bs)
    bt = workloads.make_block_table(n, bs, nb, seed=3, device="cuda")
    cache, want = (torch.full((L, nb, bs, H, d), 7.0, dtype=torch.float16, device="cuda") for _ in range(2))
    st = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    for l in range(L):
        skv.unpack_batch(cfg, [payload], [n], [bt], want, want, bs, [st], layer_begin=l, layer_count=1)
    skv.unpack(cfg, payload, cache, cache, bt, bs, st)
    assert st.item() == 0
    assert _equal(cache, want)
    gr = skv.Groups(skv.GROUP_TOKEN)
    ws = torch.empty(skv.group_workspace_size(cfg, gr), dtype=torch.uint8, device="cuda")
    skv.prepare_groups(cfg, gr, ws)
    del payload
    k = _keys(n, d)
    grouped = torch.zeros(skv.grouped_payload_size(cfg, gr), dtype=torch.uint8, device="cuda")
    skv.pack_groups(cfg, gr, k, k, tier, ws, grouped, st)
    del k
    cache.fill_(7.0)
    skv.unpack_groups(cfg, gr, ws, grouped, cache, cache, bt, bs, st)
    assert st.item() == 0
    assert _equal(cache, want)
