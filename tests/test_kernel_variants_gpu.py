"""The kernels' dispatch variants at the sizes where they can go wrong (edges
of the work split, alignment, remainders), against the oracle or a plain
float64 evaluation of the same operation."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2609_03494_amd as gp

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _say(msg):
    print(f"[variant] {msg}", flush=True)


def _offset(t: torch.Tensor, elems: int) -> torch.Tensor:
    """A contiguous copy of t whose first element lies `elems` elements into its allocation."""
    buf = torch.empty(t.numel() + elems, dtype=t.dtype, device=t.device)
    out = buf[elems:].view(t.shape)
    out.copy_(t)
    return out


def _paged(R, width, npages, gen):
    """A page table of `npages[r]` distinct pages per request in random order."""
    pool = int(sum(npages)) + 3
    perm = torch.randperm(pool, generator=gen).to(torch.int32)
    table = torch.full((R, width), -1, dtype=torch.int32)
    at = 0
    for r, P in enumerate(npages):
        table[r, :P] = perm[at:at + P]
        at += P
    return pool, table


def _state(table, num_pages, seq_lens, pool):
    i32 = lambda x: torch.as_tensor(x, dtype=torch.int32).to(DEV)
    return gp.PageState(table.to(DEV), i32(num_pages), i32(seq_lens), torch.ones(pool, dtype=torch.int32, device=DEV),
                        torch.zeros(pool, dtype=torch.int32, device=DEV), i32([0]))


# ------------------------------------------------------------------ append --

@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("layers,hq,hkv,d,offset", [(1, 8, 2, 64, 0), (3, 4, 4, 64, 1), (5, 24, 3, 128, 0),
                                                    (2, 40, 5, 128, 8), (2, 32, 8, 128, 2),
                                                    (3, 32, 8, 128, 0), (4, 24, 3, 128, 0), (7, 32, 8, 128, 0)])
def test_append_layers(dtype, layers, hq, hkv, d, offset):
    """Rows copied, summaries stepped and lengths advanced once per request,
    over one or several layers, for aligned and unaligned buffers; full, held
    and slotless requests as documented.  The copies and the fp64 EMA rounded
    once to float32 are exact."""
    _say(f"append {dtype} layers {layers} heads {hq}/{hkv} d {d} offset {offset}")
    gen = torch.Generator().manual_seed(layers * 100 + hq)
    R, M = 67, 80
    npages = [1 + r % 3 for r in range(R)]
    lens = [16 * P - 1 - (5 * r) % (16 * P) for r, P in enumerate(npages)]
    lens[3], lens[7] = 16 * npages[3], -5                       # full; held
    pool, table = _paged(R, 4, npages, gen)
    ps = _state(table, npages, lens, pool)
    randn = lambda *s: torch.randn(*s, generator=gen).to(dtype).to(DEV)
    k0, v0 = randn(layers, pool, hkv, 16, d), randn(layers, pool, hkv, 16, d)
    kc = [_offset(k0[l], offset) for l in range(layers)]
    vc = [_offset(v0[l], offset) for l in range(layers)]
    kn, vn = _offset(randn(layers, R, hkv, d), offset), _offset(randn(layers, R, hkv, d), offset)
    q = _offset(randn(layers, R, hq, d), offset)
    qs0 = torch.randn(layers, M, 2, hq, d, generator=gen)
    qstate = _offset(qs0.to(DEV), offset)
    slots = torch.randperm(M, generator=gen)[:R].to(torch.int32)
    slots[11] = M + 4                                           # no summary slot: the token still goes in
    init = torch.zeros(R, dtype=torch.uint8)
    init[5] = 1
    positions = torch.arange(R, dtype=torch.int32, device=DEV)
    gp.gp_append_step([gp.KVLayer(a, b) for a, b in zip(kc, vc)], ps, positions, kn, vn, q, slots.to(DEV),
                      init.to(DEV), qstate, 0.9, 0.999)
    torch.cuda.synchronize()
    b32 = [float(np.float32(x)) for x in (0.9, 0.999)]
    want_k, want_v, want_q = k0.cpu().clone(), v0.cpu().clone(), qs0.double().clone()
    want_len = list(lens)
    for r in range(R):
        if lens[r] < 0 or lens[r] >= 16 * npages[r]:
            continue
        pid, slot = int(table[r, lens[r] // 16]), lens[r] % 16
        want_k[:, pid, :, slot] = kn[:, r].cpu()
        want_v[:, pid, :, slot] = vn[:, r].cpu()
        want_len[r] += 1
        if int(slots[r]) < M:
            x = q[:, r].cpu().double()
            for view, b in enumerate(b32):
                prev = want_q[:, int(slots[r]), view]
                want_q[:, int(slots[r]), view] = x if int(init[r]) else b * prev + (1.0 - b) * x
    assert torch.equal(torch.stack([t.cpu() for t in kc]), want_k)
    assert torch.equal(torch.stack([t.cpu() for t in vc]), want_v)
    assert torch.equal(qstate.cpu(), want_q.float())
    assert ps.seq_lens.cpu().tolist() == want_len
    assert positions.cpu().tolist() == [r + want_len[r] - lens[r] for r in range(R)]


# ------------------------------------------------------------------ decode --
#
# Decode attention splits the batch's pages into equal runs, one per wave,
# whatever requests they belong to: requests that end inside a run, span waves,
# workgroups or whole blocks of the split's scan, empty and held ones between.

def _reference(kc, vc, table, lens, q, scale):
    """Attention of every request over its first lens[r] tokens, float64 on the CPU."""
    R, Hq, d = q.shape
    Hkv = kc.shape[1]
    G = Hq // Hkv
    out = torch.zeros(R, Hq, d, dtype=torch.float64)
    k64, v64, q64 = kc.cpu().double(), vc.cpu().double(), q.cpu().double()
    for r, m in enumerate(lens):
        if m <= 0:
            continue
        ids = table[r, :-(-m // 16)].long()
        K = k64[ids].transpose(0, 1).reshape(Hkv, -1, d)[:, :m]
        V = v64[ids].transpose(0, 1).reshape(Hkv, -1, d)[:, :m]
        z = scale * torch.matmul(q64[r].view(Hkv, G, d), K.transpose(1, 2).contiguous())
        out[r] = torch.matmul(torch.softmax(z, -1), V).view(Hq, d)
    return out


def _check(got, want, dtype, what):
    """Half a step of the output type, and float32 sums: 1e-5 of the row's largest value."""
    got, tol = got.cpu().double(), 1e-5 * want.abs().amax(-1, keepdim=True)
    if dtype == torch.bfloat16:
        tol = tol + want.abs() * 2.0 ** -8
    bad = ((got - want).abs() > tol + 1e-30) | ~torch.isfinite(got)
    assert not bad.any(), f"{what}: rows {sorted(set(bad.nonzero()[:, 0].tolist()))[:8]}"


def _decode_case(dtype, hq, hkv, d, lens, spare=0, seed=0):
    gen = torch.Generator().manual_seed(seed)
    npages = [-(-max(m, 0) // 16) + (r % 3 == 1) for r, m in enumerate(lens)]
    R, width = len(lens), max(max(npages), 1) + spare
    pool, table = _paged(R, width, npages, gen)
    # pages that nobody holds, and slots past a length, are NaN: they must not be read
    kc = torch.full((pool, hkv, 16, d), float("nan"), dtype=dtype)
    vc = kc.clone()
    for r, m in enumerate(lens):
        for p in range(-(-max(m, 0) // 16)):
            t = min(16, m - 16 * p)
            kc[table[r, p], :, :t] = torch.randn(hkv, t, d, generator=gen).to(dtype)
            vc[table[r, p], :, :t] = torch.randn(hkv, t, d, generator=gen).to(dtype)
    q = torch.randn(R, hq, d, generator=gen).to(dtype)
    kv = gp.KVLayer(kc.to(DEV), vc.to(DEV))
    return kv, table, npages, pool, q.to(DEV)


SPLITS = {
    "one_token": [1],
    "one_page_edges": [15, 16, 17, 0, 1, 33],
    "one_request": [4099],
    "a_run_each": [32] * 40,
    "mixed": [0, 700, 3, 0, 0, 2500, 16, 48, 1, 1600, 0],
    "past_a_scan_block": [(r * 37) % 50 for r in range(1100)],
    # a wide table: a workgroup each up to six pages per wave (48, or 24 with four waves), one page more, none
    "short_in_wide_table": [0, 768, 5, 384, 0, 17, 383, 1],
    "a_page_too_long": [769, 385, 40, 0, 3],
}


@pytest.mark.parametrize("name", list(SPLITS))
@pytest.mark.parametrize("spare", [5, 70, 130])    # a workgroup per request up to 64 columns, or 128 if there are many
@pytest.mark.parametrize("dtype,hq,hkv,d", [(torch.bfloat16, 8, 2, 128), (torch.bfloat16, 3, 3, 64),
                                            (torch.float32, 8, 1, 128), (torch.float32, 4, 2, 64),
                                            (torch.float32, 4, 1, 128), (torch.float32, 8, 1, 64)])
def test_decode_split(name, spare, dtype, hq, hkv, d):
    lens = SPLITS[name]
    _say(f"decode split {name} {dtype} heads {hq}/{hkv} d {d} spare table columns {spare}")
    kv, table, npages, pool, q = _decode_case(dtype, hq, hkv, d, lens, spare=spare)
    ps = _state(table, npages, lens, pool)
    ws = gp.workspace(gp.GP_OP_DECODE, len(lens), 0, hq, hkv, d, table.shape[1], dtype)
    scale = d ** -0.5
    out = torch.full_like(q, float("nan"))
    gp.gp_decode_attention(kv, ps, q, scale, out, ws)
    want = _reference(kv.k, kv.v, table, lens, q, scale)
    _check(out, want, dtype, "decode")
    # the same batch in two launches and without a workspace: the same bytes
    slots = -(-table.shape[1] // 64) + 1                    # what the static scratch is compared with
    fits = len(lens) * slots * hq * (d + 2) * 4 < 8_000_000
    for how in ("stages", "noalloc") if fits else ("stages",):
        again = torch.full_like(q, float("nan"))
        if how == "stages":
            gp.gp_decode_attention_stages(kv, ps, q, scale, again, gp.GP_DECODE_CHUNKS, ws)
            gp.gp_decode_attention_stages(kv, ps, q, scale, again, gp.GP_DECODE_MERGE, ws)
        else:
            gp.gp_decode_attention_noalloc(kv, ps, q, scale, again)
        torch.cuda.synchronize()
        assert torch.equal(again.view(torch.uint8), out.view(torch.uint8)), how
    # held requests keep their place: nobody else's output changes
    held = [r for r in range(0, len(lens), 3) if lens[r] > 0]
    for r in held:
        ps.seq_lens[r] = -lens[r] - 1
    again = torch.full_like(q, 7.0)
    gp.gp_decode_attention(kv, ps, q, scale, again, ws)
    torch.cuda.synchronize()
    keep = torch.tensor([r not in held for r in range(len(lens))], device=DEV)
    assert torch.equal(again[keep], out[keep]) and bool((again[~keep] == 7.0).all())


def _attend(kv, table, npages, pool, lens, q, hq, hkv, d, dtype, scale):
    ps = _state(table, npages, lens, pool)
    ws = gp.workspace(gp.GP_OP_DECODE, len(lens), 0, hq, hkv, d, table.shape[1], dtype)
    out = torch.full_like(q, 7.0)
    gp.gp_decode_attention(kv, ps, q, scale, out, ws)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("spare", [2, 130])
@pytest.mark.parametrize("hq,hkv,d", [(3, 3, 64), (8, 4, 64), (2, 2, 128), (4, 2, 128)])
def test_decode_weights_in_float32(hq, hkv, d, spare):
    """One and two query heads per KV head: P.V keeps the weights' float32 bits.
    Three tokens, weights w0 = 1, wA and wB nearly equal, values 0, 1, -1: the
    output (wA - wB) / (1 + wA + wB) is of the order of 1e-4, where a weight
    rounded to 17 bits shows.  Scores are exact in float32 (few-bit factors), so
    what is left is an exp2 unit of each weight (2^-23 together) and the output's
    rounding."""
    _say(f"float32 weights heads {hq}/{hkv} d {d} spare {spare}")
    gen = torch.Generator().manual_seed(d + hq)
    R, dtype, G = 48, torch.bfloat16, hq // hkv
    kv, table, npages, pool, q = _decode_case(dtype, hq, hkv, d, [3] * R, spare=spare)
    k, v = kv.k.cpu(), kv.v.cpu()
    q = torch.randint(-4, 5, (R, hq, d), generator=gen).to(dtype) / 8
    q[..., 0] = torch.randint(1, 9, (R, hq), generator=gen).to(dtype) / 16
    for r in range(R):
        pid = int(table[r, 0])
        base = torch.randint(-4, 5, (hkv, d), generator=gen).float() / 8
        base[:, 0] = 1.0
        k[pid, :, 0] = 0
        k[pid, :, 1] = (base - 2 * torch.sign((base * q[r, ::G].float()).sum(-1, keepdim=True)) * base).to(dtype)
        k[pid, :, 2] = k[pid, :, 1]
        k[pid, :, 2, 0] = k[pid, :, 1, 0] * (1 + 2.0 ** -7)
        v[pid, :, 0], v[pid, :, 1], v[pid, :, 2] = 0, 1, -1
    kv, q = gp.KVLayer(k.to(DEV), v.to(DEV)), q.to(DEV)
    scale = 0.125
    got = _attend(kv, table, npages, pool, [3] * R, q, hq, hkv, d, dtype, scale).cpu().double()
    want = _reference(kv.k, kv.v, table, [3] * R, q, scale)
    bad = (got - want).abs() > want.abs() * 2.0 ** -8 + 2.0 ** -22
    assert not bad.any(), f"{int(bad.any(-1).sum())} of {R * hq} rows, worst {float((got - want).abs().max()):.2e}"


@pytest.mark.parametrize("hq,hkv,d", [(12, 12, 64), (32, 8, 128), (16, 2, 128)])
def test_decode_f32_error(hq, hkv, d):
    """Large scores (keys of four times the norm) in float32: the output is off
    by no more than twice what one rounding of every score (in log2 units) and
    weight to float32 costs -- the score's own sum and its scaling lose about as
    much again."""
    _say(f"float32 error heads {hq}/{hkv} d {d}")
    lens, dtype, scale = [500 + 640 * r for r in range(8)], torch.float32, d ** -0.5
    kv, table, npages, pool, q = _decode_case(dtype, hq, hkv, d, lens, seed=5)
    kv.k.mul_(4)
    got = _attend(kv, table, npages, pool, lens, q, hq, hkv, d, dtype, scale).cpu().double()
    want = _reference(kv.k, kv.v, table, lens, q, scale)
    once = torch.zeros_like(want)
    k, v, G = kv.k.cpu().double(), kv.v.cpu().double(), hq // hkv
    s32 = float(np.float32(scale)) * 1.4426950408889634
    for r, m in enumerate(lens):
        ids = table[r, :-(-m // 16)].long()
        K, V = (t[ids].transpose(0, 1).reshape(hkv, -1, d)[:, :m] for t in (k, v))
        z = (s32 * torch.matmul(q[r].cpu().double().view(hkv, G, d), K.transpose(1, 2).contiguous())).float()
        w = torch.exp2(z - z.amax(-1, keepdim=True)).double()
        once[r] = (torch.matmul(w, V) / w.sum(-1, keepdim=True)).view(hq, d)
    err, bar = float((got - want).norm() / want.norm()), float((once - want).norm() / want.norm())
    assert err <= 2 * bar, f"error {err:.2e}, one rounding {bar:.2e}"


@pytest.mark.parametrize("spare", [2, 130])
@pytest.mark.parametrize("dtype,hq,hkv,d", [(torch.bfloat16, 3, 3, 64), (torch.bfloat16, 8, 2, 128), (torch.float32, 2, 2, 64),
                                            (torch.float32, 4, 1, 128), (torch.float32, 8, 1, 64)])
def test_decode_small_weights(dtype, hq, hkv, d, spare):
    """A weight of 2^-130 beside one of 1 whose value is zero: the result is that
    weight times its value (a subnormal weight has 2^-150 of absolute error, here
    2^-20 of the result), with both tokens in one page and in two of them."""
    _say(f"small weights {dtype} heads {hq}/{hkv} d {d} spare {spare}")
    lens = [2, 17]
    kv, table, npages, pool, q = _decode_case(dtype, hq, hkv, d, lens, spare=spare)
    kv.k.zero_(), kv.v.zero_(), q.zero_()
    q[..., 0] = 1.0
    scale = 1.0 / 1.4426950408889634
    for r, m in enumerate(lens):
        kv.k[int(table[r, 0]), :, :, 0] = -600.0                # 2^-600: zero beside the others
        kv.k[int(table[r, 0]), :, 0, 0] = 0.0
        kv.k[int(table[r, (m - 1) // 16]), :, (m - 1) % 16, 0] = -130.0
        kv.v[int(table[r, (m - 1) // 16]), :, (m - 1) % 16] = 2.0 ** 100
    got = _attend(kv, table, npages, pool, lens, q, hq, hkv, d, dtype, scale).cpu().double()
    # the float32 scale moves 2^-130 by 130 of its roundings at most
    assert bool(((got / 2.0 ** -30 - 1).abs() < 2.0 ** -16).all()), got.flatten()[:4]


@pytest.mark.parametrize("spare", [2, 130])
@pytest.mark.parametrize("hq,hkv,d", [(3, 3, 64), (8, 2, 128)])
def test_decode_division(hq, hkv, d, spare):
    """The output is the sum divided by the weights' sum, rounded once: seven
    equal weights and values whose sum is seven times the midpoint of two
    bfloat16 numbers give the even one (the product with a rounded reciprocal
    misses the midpoint)."""
    _say(f"division heads {hq}/{hkv} d {d} spare {spare}")
    dtype, lens = torch.bfloat16, [7]
    kv, table, npages, pool, q = _decode_case(dtype, hq, hkv, d, lens, spare=spare)
    mid = (257 + 2 * torch.arange(d) % 256).float() / 256                 # nine significant bits
    want = mid.to(dtype)
    pid = int(table[0, 0])
    kv.k.zero_()
    kv.v.zero_()
    high = (7 * mid).to(dtype)
    kv.v[pid, :, 0], kv.v[pid, :, 3] = high.to(DEV), (7 * mid - high.float()).to(dtype).to(DEV)
    assert torch.equal(kv.v[pid, 0].cpu().float().sum(0), 7 * mid)
    got = _attend(kv, table, npages, pool, lens, q, hq, hkv, d, dtype, d ** -0.5).cpu()
    assert torch.equal(got, want.expand_as(got)), (got != want).sum()


@pytest.mark.parametrize("spare", [2, 130])
@pytest.mark.parametrize("dtype,hq,hkv,d", [(torch.bfloat16, 3, 3, 64), (torch.bfloat16, 8, 2, 128), (torch.float32, 4, 2, 64),
                                            (torch.float32, 8, 1, 128)])
def test_decode_nan_scores(dtype, hq, hkv, d, spare):
    """A NaN key gives a zero output, however the batch's split cuts its request
    (one wave, several waves of a workgroup, several workgroups); the others'
    outputs are theirs."""
    _say(f"NaN scores {dtype} heads {hq}/{hkv} d {d} spare {spare}")
    lens = [5, 16, 17, 300, 40, 1000, 900, 2000 if spare > 64 else 1, 33]
    kv, table, npages, pool, q = _decode_case(dtype, hq, hkv, d, lens, spare=spare)
    scale = d ** -0.5
    want = _reference(kv.k, kv.v, table, lens, q, scale)
    for r in (0, 2, 3, 5, 7):
        t = lens[r] * 2 // 3
        kv.k[int(table[r, t // 16]), :, t % 16, 3] = float("nan")
        want[r] = 0.0
    got = _attend(kv, table, npages, pool, lens, q, hq, hkv, d, dtype, scale)
    _check(got, want, dtype, "decode beside NaN")


@pytest.mark.parametrize("spare", [2, 130])
@pytest.mark.parametrize("hq,hkv,d", [(3, 3, 64), (4, 2, 128)])
def test_decode_infinite_values(hq, hkv, d, spare):
    """An infinite value in a resident slot gives that infinity (one and two
    query heads per KV head, whose weights are one float32 number each)."""
    _say(f"infinite values heads {hq}/{hkv} d {d} spare {spare}")
    lens, dtype = [40, 700, 3, 1000, 16], torch.bfloat16
    kv, table, npages, pool, q = _decode_case(dtype, hq, hkv, d, lens, spare=spare)
    want = _reference(kv.k, kv.v, table, lens, q, d ** -0.5)
    for r, m in enumerate(lens):
        t = (7 * r + 2) % m
        kv.v[int(table[r, t // 16]), :, t % 16, 5] = float("inf")
        kv.v[int(table[r, t // 16]), :, t % 16, 9] = -float("inf")
    got = _attend(kv, table, npages, pool, lens, q, hq, hkv, d, dtype, d ** -0.5)
    assert bool((got[..., 5] == float("inf")).all()) and bool((got[..., 9] == -float("inf")).all())
    got[..., [5, 9]] = want[..., [5, 9]].to(DEV, dtype)
    _check(got, want, dtype, "decode beside infinite values")


@pytest.mark.parametrize("spare", [2, 130])
@pytest.mark.parametrize("offset", [1, 2])
@pytest.mark.parametrize("dtype,hq,hkv,d", [(torch.float32, 4, 2, 64), (torch.float32, 4, 1, 128), (torch.float32, 8, 1, 64),
                                            (torch.bfloat16, 8, 2, 128), (torch.bfloat16, 3, 3, 64)])
def test_decode_unaligned(dtype, hq, hkv, d, offset, spare):
    """Buffers one or two elements into their allocations (bfloat16 pools excepted)
    give the bytes of aligned ones: decode attention, and a step with a token."""
    _say(f"unaligned {dtype} heads {hq}/{hkv} d {d} offset {offset} spare {spare}")
    lens = [1, 40, 0, 700, 16, 77, 1500 if spare > 64 else 33]
    R, scale = len(lens), d ** -0.5
    kv, table, npages, pool, q = _decode_case(dtype, hq, hkv, d, lens, spare=spare)
    gen = torch.Generator().manual_seed(3)
    rand = lambda *s: torch.randn(*s, generator=gen).to(dtype).to(DEV)
    q_pre, k_new, v_new = rand(R, hq, d), rand(R, hkv, d), rand(R, hkv, d)
    qs = torch.randn(R, 2, hq, d, generator=gen).to(DEV)
    slots, init = torch.arange(R, dtype=torch.int32, device=DEV), torch.zeros(R, dtype=torch.uint8, device=DEV)
    n = gp.gp_workspace_bytes(gp.GP_OP_DECODE, R, 0, hq, hkv, d, table.shape[1], dtype)
    results = []
    for off in (0, offset):
        at = lambda t: _offset(t, off)
        pool_at = at if dtype == torch.float32 else torch.clone
        layer = gp.KVLayer(pool_at(kv.k), pool_at(kv.v))
        ps = _state(table, npages, lens, pool)
        ws = torch.zeros(n + 16, dtype=torch.uint8, device=DEV)[4 * off:4 * off + n]
        out, out2, qstate = at(torch.full_like(q, 7.0)), at(torch.full_like(q, 7.0)), at(qs)
        gp.gp_decode_attention(layer, ps, at(q), scale, out, ws)
        gp.gp_decode_step(layer, ps, at(q), at(q_pre), scale, out2, slots, init, qstate, 0.9, 0.999, ws, at(k_new),
                          at(v_new), torch.zeros(R, dtype=torch.int32, device=DEV))
        torch.cuda.synchronize()
        results.append([out, out2, qstate, layer.k, layer.v, ps.seq_lens])
    for a, b in zip(*results):
        assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))
    _check(results[1][0], _reference(kv.k, kv.v, table, lens, q, scale), dtype, "decode")


# lengths whose new token opens a page (16 n): at a request's first page, at the first
# page of a wave's run and of a workgroup, beside full (F), held (H) and empty requests
STEPS = {
    "opens_pages": [0, 16, 32, 256, 512, 768, 15, 31, 1, 480, "F48", "H64", 33],
    "one_long": [2048],
    "runs_of_two_pages": [32, "F32", 32, 32, "H32", 31, 32, 32, 0, 32] * 5,
    "long_and_short": [1600, 5, "F16", 2047, "H700", 0, 1023, 16],
}


@pytest.mark.parametrize("name", list(STEPS))
@pytest.mark.parametrize("spare", [2, 140])
@pytest.mark.parametrize("repeat", [1, 9])
@pytest.mark.parametrize("dtype,hq,hkv,d", [(torch.bfloat16, 3, 3, 64), (torch.bfloat16, 8, 4, 64), (torch.bfloat16, 16, 4, 64),
                                            (torch.bfloat16, 16, 2, 64), (torch.bfloat16, 4, 4, 128), (torch.bfloat16, 8, 2, 128),
                                            (torch.float32, 4, 2, 64), (torch.float32, 8, 1, 64), (torch.float32, 2, 2, 128),
                                            (torch.float32, 8, 1, 128)])
def test_step_token_split(name, spare, repeat, dtype, hq, hkv, d):
    """gp_decode_step with a token in every form of the decode kernel (a workgroup of
    four or eight waves per request, equal runs): the cache, lengths and summaries
    of gp_append_step bit for bit, outputs of decode attention after it, and both
    against float64."""
    spec = STEPS[name] * (repeat if len(STEPS[name]) < 20 else 1)
    full, held = ([str(m)[0] == c for m in spec] for c in "FH")
    lens = [int(m[1:]) if isinstance(m, str) else m for m in spec]
    if repeat > 1:                                             # (512 pairs: four waves per request at d 64)
        spec_n = -(-512 // hkv)
        while len(lens) < spec_n and max(lens) < 1000:
            lens, full, held = lens + lens, full + full, held + held
    _say(f"step {name} x{repeat} {dtype} heads {hq}/{hkv} d {d} spare {spare}: {len(lens)} requests")
    R, scale = len(lens), d ** -0.5
    gen = torch.Generator().manual_seed(R + d)
    # a page for the token, but for the full ones
    npages = [m // 16 if f else m // 16 + 1 for m, f in zip(lens, full)]
    width = max(npages) + spare
    pool, table = _paged(R, width, npages, gen)
    kc = torch.full((pool, hkv, 16, d), float("nan"), dtype=dtype)
    vc = kc.clone()
    for r, m in enumerate(lens):
        for p in range(-(-m // 16)):
            t = min(16, m - 16 * p)
            kc[table[r, p], :, :t] = torch.randn(hkv, t, d, generator=gen).to(dtype)
            vc[table[r, p], :, :t] = torch.randn(hkv, t, d, generator=gen).to(dtype)
    rand = lambda *s: torch.randn(*s, generator=gen).to(dtype).to(DEV)
    q, q_pre, k_new, v_new = rand(R, hq, d), rand(R, hq, d), rand(R, hkv, d), rand(R, hkv, d)
    qs = torch.randn(R + 3, 2, hq, d, generator=gen).to(DEV)
    slots = torch.randperm(R + 3, generator=gen)[:R].to(torch.int32).to(DEV)
    init = (torch.arange(R) % 5 == 4).to(torch.uint8).to(DEV)
    dev_lens = [-m - 1 if h else m for m, h in zip(lens, held)]
    n = gp.gp_workspace_bytes(gp.GP_OP_DECODE, R, 0, hq, hkv, d, width, dtype)
    results = []
    for fused in (True, False):
        kv = gp.KVLayer(kc.to(DEV), vc.to(DEV))
        ps, pos = _state(table, npages, dev_lens, pool), torch.arange(R, dtype=torch.int32, device=DEV)
        out, qstate = torch.full_like(q, 7.0), qs.clone()
        ws = torch.zeros(n, dtype=torch.uint8, device=DEV)
        if fused:
            gp.gp_decode_step(kv, ps, q, q_pre, scale, out, slots, init, qstate, 0.9, 0.999, ws, k_new, v_new, pos)
        else:
            gp.gp_append_step([kv], ps, pos, k_new.unsqueeze(0), v_new.unsqueeze(0), q_pre.unsqueeze(0), slots, init,
                              qstate.unsqueeze(0), 0.9, 0.999)
            gp.gp_decode_attention(kv, ps, q, scale, out, ws)
        torch.cuda.synchronize()
        results.append([kv.k, kv.v, qstate, pos, ps.seq_lens, out])
    for what, a, b in zip(("keys", "values", "summaries", "positions", "lengths"), *results):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), what
    k_, v_, _, _, new_lens, out = results[0]
    assert new_lens.cpu().tolist() == [m if f or h else m + 1 for m, f, h in zip(dev_lens, full, held)]
    assert bool((out[torch.tensor(held, device=DEV)] == 7.0).all())
    ref_lens = [0 if h else max(m, 0) for m, h in zip(new_lens.cpu().tolist(), held)]
    want = _reference(k_, v_, table, ref_lens, q, scale)
    for got in (out, results[1][5]):
        got[torch.tensor(held, device=DEV)] = 0.0
        _check(got, want, dtype, "step")


@pytest.mark.parametrize("hq,hkv,d", [(16, 2, 128), (4, 4, 64), (8, 2, 64)])
@pytest.mark.parametrize("prefix", [1, 5, 70])
def test_decode_shared_split(hq, hkv, d, prefix):
    """Members with the whole prefix, with one page of it replaced (first,
    middle, last), shorter than the prefix, exactly as long, one token longer,
    held; and requests outside the group."""
    _say(f"shared decode split heads {hq}/{hkv} d {d} prefix {prefix}")
    dtype, P = torch.bfloat16, prefix
    tails = [40, 1, 0, 17, 300, 33, 64, 2000, 16]
    lens = [16 * P + t for t in tails] + [max(16 * P - 3, 1), 77]
    kv, table, npages, pool, q = _decode_case(dtype, hq, hkv, d, lens, spare=3, seed=prefix)
    R = len(lens)
    k, v = kv.k.cpu(), kv.v.cpu()
    for r in range(1, R - 1):                              # the group: all but the last request
        keep = {3: 0, 4: P // 2, 5: P - 1}.get(r, -1)      # a page of its own
        for p in range(min(P, -(-lens[r] // 16))):
            if p != keep:
                table[r, p] = table[0, p]
    kv = gp.KVLayer(k.to(DEV), v.to(DEV))
    lens[6] = -lens[6] - 1                                 # held
    ps = _state(table, npages, lens, pool)
    scale = d ** -0.5
    ws = gp.workspace(gp.GP_OP_DECODE, R, 0, hq, hkv, d, table.shape[1], dtype)
    out = torch.full_like(q, 7.0)
    gp.gp_decode_attention_shared(kv, ps, q, scale, out, [(0, R - 1, P)], ws)
    torch.cuda.synchronize()
    want = _reference(kv.k, kv.v, table, lens, q, scale)
    assert bool((out[6] == 7.0).all())
    out[6] = 0.0
    _check(out, want, dtype, "shared decode")


# ------------------------------------------------------------------ decide --

@pytest.mark.parametrize("events", [1, 7, 64, 513, 1500, 2048])
@pytest.mark.parametrize("stack", ["ample", "exact", "short", "none"])
def test_decide_pages_in_list_order(events, stack):
    """Pages are handed out in list order, whether the stack covers everybody
    (prefix sum) or not (one request after the other): grows get the top pages
    in order, then fall back, shared pages are replaced, and the reserve holds.
    The expectation is the sequential rule itself."""
    _say(f"decide {events} events, stack {stack}")
    gen = torch.Generator().manual_seed(events)
    hkv, d, width, reserve = 1, 64, 4, 2
    npages = [1 + (r * 7) % 3 for r in range(events)]
    want = [bool((r * 5) % 4 < 2) for r in range(events)]
    shared = [(r % 6 == 1) and npages[r] > 1 for r in range(events)]
    pops = sum(1 if w else s for w, s in zip([w or p == 1 for w, p in zip(want, npages)], shared))
    free = {"ample": pops + reserve + 5, "exact": pops + reserve, "short": pops // 2 + reserve, "none": reserve}[stack]
    pool, table = _paged(events, width, npages, gen)
    pool += free
    refs = torch.zeros(pool, dtype=torch.int32)
    for r in range(events):
        refs[table[r, :npages[r]].long()] = 1
        if shared[r]:
            refs[int(table[r, 0])] = 2
    stack_ids = torch.arange(pool - free, pool, dtype=torch.int32)
    free_list = torch.zeros(pool, dtype=torch.int32)
    free_list[:free] = stack_ids
    i32 = lambda x: torch.as_tensor(x, dtype=torch.int32).to(DEV)
    ps = gp.PageState(table.to(DEV), i32(npages), i32([16 * p for p in npages]), refs.to(DEV), free_list.to(DEV),
                      i32([free]))
    kv = gp.KVLayer(*(torch.randn(pool, hkv, 16, d, generator=gen).to(torch.bfloat16).to(DEV) for _ in range(2)))
    order = torch.randperm(events, generator=gen).to(torch.int32)
    counts = torch.tensor([[[[6, 5] if want[int(r)] else [5, 6]] for r in order]], dtype=torch.int32).to(DEV)
    scores = torch.rand(1, events, hkv, (width - 1) * 16, generator=gen).to(DEV)
    dec, delta = torch.full((events,), -1, dtype=torch.int32, device=DEV), torch.zeros(events, device=DEV)
    counters = torch.zeros(4, dtype=torch.int64, device=DEV)
    ws = gp.workspace(gp.GP_OP_APPLY, events, events, 1, hkv, d, width, torch.bfloat16)
    gp.gp_boundary_apply([kv], ps, order.to(DEV), counts, scores, gp.Params(reserve_pages=reserve), dec, delta,
                         counters, ws)
    torch.cuda.synchronize()
    top, expect, want_table, tally = free, [], table.clone(), [0] * 4
    for r in order.tolist():
        P = npages[r]
        if (want[r] or P == 1) and top > reserve:
            top -= 1
            want_table[r, P] = stack_ids[top]
            expect.append(gp.GP_GROW)
        elif P == 1 or (shared[r] and top < 1):
            expect.append(gp.GP_PREEMPT)
        else:
            if shared[r]:
                top -= 1
                want_table[r, 0] = stack_ids[top]
            expect.append(gp.GP_FALLBACK if want[r] else gp.GP_COMPRESS)
        tally[expect[-1]] += 1
    assert dec.cpu().tolist() == expect
    assert torch.equal(ps.page_table.cpu(), want_table)
    assert int(ps.free_count) == top and counters.cpu().tolist() == tally


@pytest.mark.parametrize("policy", [gp.GP_POLICY_GROWPAGE, gp.GP_POLICY_SHRINK])
@pytest.mark.parametrize("pages,shared", [(3, "all"), (65, "all"), (129, "prefix 128"), (130, "every 3rd"), (512, "all"),
                                          (513, "every 3rd"), (600, "prefix 513"), (1025, "all"), (1600, "every 3rd"),
                                          (2100, "prefix 1537")])
def test_decide_long_shared_rows(pages, shared, policy):
    """Shared pages over several blocks of a row (64 pages a ballot, 512 a wave,
    1024 a selection count): private pages in order of the logical page, the old
    references dropped, pages nobody holds any more back on the stack by id, and
    a shrink's last page dropped; two requests of the same row, one beside them
    that stays."""
    _say(f"decide {pages} pages, shared: {shared}, policy {policy}")
    gen = torch.Generator().manual_seed(pages)
    hkv, d, R, shrink = 1, 64, 3, policy == gp.GP_POLICY_SHRINK
    width = pages + 3
    kind, _, num = shared.partition(" ")
    is_shared = [kind == "all" or (kind == "prefix" and j < int(num)) or (kind == "every" and j % 3 == 1)
                 for j in range(pages)]
    pool = 6 * pages + 40
    perm = torch.randperm(pool, generator=gen).to(torch.int32)
    table = torch.full((R, width), -1, dtype=torch.int32)
    refs = torch.zeros(pool, dtype=torch.int32)
    at = 0
    for j in range(pages):
        for r in range(R):
            if r and is_shared[j]:
                table[r, j] = table[0, j]
            else:
                table[r, j], at = perm[at], at + 1
            refs[int(table[r, j])] += 1
    free = pool - at
    free_list = torch.zeros(pool, dtype=torch.int32)
    free_list[:free] = perm[at:]
    i32 = lambda x: torch.as_tensor(x, dtype=torch.int32).to(DEV)
    lens = [16 * pages, 16 * pages, 16 * pages - 5]           # the last one is not at a boundary
    ps = gp.PageState(table.to(DEV), i32([pages] * R), i32(lens), refs.to(DEV), free_list.to(DEV), i32([free]))
    kc = torch.randn(pool, hkv, 16, d, generator=gen).to(torch.bfloat16).to(DEV)
    kv = gp.KVLayer(kc, kc.clone())
    order = [1, 0]
    counts = torch.tensor([[[[5, 60]]] * 2], dtype=torch.int32).to(DEV)
    scores = torch.rand(1, 2, hkv, (width - 1) * 16, generator=gen).to(DEV)
    dec, delta = torch.full((2,), -1, dtype=torch.int32, device=DEV), torch.zeros(2, device=DEV)
    counters = torch.zeros(4, dtype=torch.int64, device=DEV)
    ws = gp.workspace(gp.GP_OP_APPLY, R, 2, hkv, hkv, d, width, torch.bfloat16)
    gp.gp_boundary_apply([kv], ps, i32(order), counts, scores,
                         gp.Params(policy=policy, min_capacity_pages=2, shrink_threshold=0.0), dec, delta, counters, ws)
    torch.cuda.synchronize()
    want, want_refs, top = table.clone(), refs.clone(), free
    keep = pages - 1 if shrink else pages
    released = []
    for r in order:
        fresh = [j for j in range(keep) if is_shared[j]]
        for j in fresh + ([pages - 1] if shrink else []):
            old = int(table[r, j])
            want_refs[old] -= 1
            if want_refs[old] == 0:
                released.append(old)
        for k, j in enumerate(fresh):
            want[r, j] = free_list[top - 1 - k]
            want_refs[int(want[r, j])] = 1
        top -= len(fresh)
        if shrink:
            want[r, pages - 1] = -1
    assert dec.cpu().tolist() == [gp.GP_SHRINK if shrink else gp.GP_COMPRESS] * 2
    assert torch.equal(ps.page_table.cpu(), want)
    assert torch.equal(ps.refcount.cpu(), want_refs)
    assert int(ps.free_count) == top + len(released)
    assert ps.free_list.cpu()[top:top + len(released)].tolist() == sorted(released)
