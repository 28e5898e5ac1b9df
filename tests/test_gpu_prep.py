"""Restoring groups of small tensors, whose headers, counts and scans are one launch, and groups just past that size (32
tiles of 4096 elements), against the oracle: same values, same refusal of a blob whose bitmap and header disagree.  And
groups of so many tiles that a wave counts several, across the borders of tensors."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2406_11257_amd as X
from gpu_util import to_dev

pytestmark = pytest.mark.gpu
f32 = np.float32


@pytest.mark.parametrize("flags", [0, X.EXCP_FLAG_NO_W2M])
@pytest.mark.parametrize("largest", [32 * 4096, 32 * 4096 + 1])
def test_small_groups_and_the_first_larger_one(largest, flags):
    sizes = [largest, 1, 64, 4096, 4097, 4 * 4096, 5 * 4096 + 1, 29 * 4096 + 63]
    ctx = X.Context(largest, sum(sizes))
    cases, dev = [], []
    for n in sizes:
        g = np.random.default_rng(n)
        Wp = (g.standard_normal(n) * 0.02).astype(f32)
        W = (Wp + g.laplace(0, 1e-4, n)).astype(f32)
        m = (g.standard_normal(n) * 5e-5).astype(f32)
        v = (m.astype(np.float64) ** 2 * g.lognormal(0, 1, n) + 1e-16).astype(f32)
        blob = O.compress_step(Wp, W, m, v, 5e-5, 2.0, 4, 2, flags=flags).blob
        out = [torch.full((n,), 3.0, device="cuda") for _ in range(3)]
        cases.append((Wp, blob, out))
        dev.append([to_dev(Wp), torch.from_numpy(np.frombuffer(blob, np.uint8).copy()).cuda(), len(blob), n, *out])
    # a kept element more than the header says, in the second last bit of the last tile's bitmap
    bad = np.frombuffer(cases[-1][1], np.uint8).copy()
    at = 80 + 12 * 16 + (sizes[-1] - 2) // 8
    bad[at] ^= 1 << ((sizes[-1] - 2) % 8)
    print(largest, flags, flush=True)
    for damaged in (False, True):
        if damaged:
            dev[-1][1] = torch.from_numpy(bad).cuda()
            for o in cases[-1][2]:
                o.fill_(3.0)
        ctx.excp_decompress_tensors([tuple(d) for d in dev])
        rc, stats = ctx.excp_collect(check=False)
        assert rc == (X.EXCP_E_BLOB if damaged else 0)
        for i, ((Wp, blob, out), st) in enumerate(zip(cases, stats)):
            if damaged and i == len(cases) - 1:
                assert st.status == X.EXCP_E_BLOB and all(torch.all(o == 3.0) for o in out)
                continue
            assert st.status == 0
            for got, want in zip(out, O.decompress_step(Wp, blob)):
                assert got.cpu().numpy().tobytes() == want.tobytes()
    ctx.close()


def test_waves_that_count_several_tiles_across_tensors():
    # 256 compute units count 8192 tiles at once.  About twice and three times as many tiles, in tensors of 1 to 199, the
    # borders anywhere in a wave's range; then fewer than there are waves.
    for sizes in ([4096 * (1 + (37 * i) % 199) - (i % 3) * 17 for i in range(170)], [4096 * (1 + (53 * i) % 97) - (i % 5) for i in range(500)],
                  [33 * 4096 + 1, 70_000, 5, 4096 * 9]):
        ctx = X.Context(max(sizes), sum(sizes))
        gen = torch.Generator(device="cuda")
        gen.manual_seed(len(sizes))
        comp, dec, outs = [], [], []
        for n in sizes:
            Wp = torch.empty(n, device="cuda").normal_(0, 0.02, generator=gen)
            W = Wp + torch.empty(n, device="cuda").normal_(0, 1e-4, generator=gen)
            m = torch.empty(n, device="cuda").normal_(0, 5e-5, generator=gen)
            v = m * m * torch.empty(n, device="cuda").normal_(generator=gen).exp() + 1e-16
            comp.append((Wp, W, m, v, torch.zeros(X.excp_blob_bound(n, 4), dtype=torch.uint8, device="cuda"), torch.zeros_like(Wp)))
        print(len(sizes), sum((n + 4095) // 4096 for n in sizes), flush=True)
        ctx.excp_compress_tensors(comp, 5e-5, 2.0, 4, 1, 0)
        rc, stats = ctx.excp_collect(check=False)
        assert rc == 0
        for moments in (True, False):
            outs = [[torch.full((n,), 3.0, device="cuda") if k == 0 or moments else None for k in range(3)] for n in sizes]
            ctx.excp_decompress_tensors([(c[0], c[4], int(st.blob_bytes), n, *o) for c, st, n, o in zip(comp, stats, sizes, outs)])
            rc, _ = ctx.excp_collect(check=False)
            assert rc == 0
            # every tensor's weights as the compress call left them (its counts come from the mask pass), and some tensors
            # in full against the oracle
            assert all(torch.equal(o[0], c[5]) for c, o in zip(comp, outs))
            for i in range(0, len(sizes), 19) if moments else ():
                ref = O.decompress_step(comp[i][0].cpu().numpy(), comp[i][4][:stats[i].blob_bytes].cpu().numpy().tobytes())
                for got, want in zip(outs[i], ref):
                    assert got.cpu().numpy().tobytes() == want.tobytes()
        ctx.close()
