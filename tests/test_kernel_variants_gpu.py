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
                                                    (2, 40, 5, 128, 8), (2, 32, 8, 128, 2)])
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
