"""Groups of small tensors (k_small.hip) against the oracle, blob for blob and with W_hat: sizes from none to the most elements
a workgroup holds and one more (which takes the general kernels), every code width, the weights' storages, ties, values many
binary orders apart, subnormal ones, crowded cells, the error paths, and W_hat written over W_prev."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2406_11257_amd as X

pytestmark = pytest.mark.gpu
f32 = np.float32
KIND = {0: torch.float32, X.EXCP_FLAG_W_F16: torch.float16, X.EXCP_FLAG_W_BF16: torch.bfloat16}


def draw(n, seed, kind, flags=0):
    g = np.random.default_rng(seed)
    scale = 1e-3 if flags & 0x30 else 1e-4
    if kind == "spread":
        d = g.laplace(0, scale, n)
    elif kind == "tied":
        d = g.integers(-4, 5, n) * 2.0 ** -10 + np.where(g.random(n) < 0.05, g.normal(0, 1e-3, n), 0.0)
    elif kind == "far apart":               # more binary orders than 128-bit sums hold, subnormal values among them
        d = 2.0 ** g.uniform(-140, -5, n) * g.choice([-1.0, 1.0], n)
    elif kind == "crowded":                 # nearly all in one cell
        d = np.where(g.random(n) < 0.02, g.uniform(-1, 1, n), 1e-4 * (1 + 1e-5 * g.standard_normal(n)))
    else:                                   # "equal"
        d = np.full(n, 2.0 ** -9)
    Wp = np.zeros(n, f32) if kind == "far apart" else O.narrow((g.standard_normal(n) * 0.02).astype(f32), flags)
    Wp = O.narrow(np.asarray(Wp, f32), flags) if kind == "far apart" else Wp
    W = O.narrow((O.widen(Wp, flags) + d.astype(f32)).astype(f32), flags)
    m = (g.standard_normal(n) * 5e-5).astype(f32)
    if kind == "far apart": m = (2.0 ** g.uniform(-140, 0, n) * g.choice([-1.0, 1.0], n)).astype(f32)
    v = (m.astype(np.float64) ** 2 * g.lognormal(0, 1, n) + 1e-16).astype(f32)
    return Wp, W, m, v


def put_w(a, flags):
    return torch.from_numpy(np.ascontiguousarray(a).view(f32 if not flags & 0x30 else np.int16)).cuda().view(KIND[flags & 0x30])


def run(ctx, cases, nbits, iters, alpha, beta, flags, in_place=False):
    items, outs = [], []
    for Wp, W, m, v in cases:
        n = m.size
        wp = put_w(Wp, flags)
        out = wp if in_place else torch.zeros_like(wp)
        items.append((wp, put_w(W, flags), torch.from_numpy(m).cuda(), torch.from_numpy(v).cuda(),
                      torch.full((X.excp_blob_bound(n, nbits),), 0xAB, dtype=torch.uint8, device="cuda"), out))
        outs.append(out)
    ctx.excp_compress_tensors(items, alpha, beta, nbits, iters, flags)
    rc, stats = ctx.excp_collect(check=False)
    return rc, stats, items, outs


def check(ctx, cases, nbits, iters, alpha=5e-5, beta=2.0, flags=0, in_place=False):
    rc, stats, items, outs = run(ctx, cases, nbits, iters, alpha, beta, flags, in_place)
    assert rc == 0
    for c, st, it, out in zip(cases, stats, items, outs):
        ref = O.compress_step(*c, alpha, beta, nbits, iters, flags=flags)
        blob = it[4][:st.blob_bytes].cpu().numpy().tobytes()
        assert (st.n_w, st.n_o) == (ref.n_w, ref.n_o)
        assert blob == ref.blob
        assert f32(st.median_abs_dw).tobytes() == f32(ref.median).tobytes() and st.abs_sum_m == ref.abs_sum_m
        np.testing.assert_allclose([st.obj_w, st.obj_m, st.obj_v], [ref.obj[k] for k in "wmv"], rtol=1e-12)        # (8192 non-negative terms in fp64)
        want = O.decompress_step(c[0], ref.blob)[0]
        assert out.view(torch.int16 if flags & 0x30 else torch.int32).cpu().numpy().tobytes() == np.ascontiguousarray(want).tobytes()


@pytest.fixture(scope="module")
def ctx():
    c = X.Context(20_000, 400_000)
    yield c
    c.close()


SIZES = [0, 1, 2, 63, 64, 65, 127, 1000, 4095, 4096, 4097, 8191, 8192]


@pytest.mark.parametrize("kind", ["spread", "tied", "far apart", "crowded", "equal"])
@pytest.mark.parametrize("nbits", [2, 4, 6, 7, 8])
def test_sizes_widths_and_values(ctx, kind, nbits):
    for alpha, beta, iters in ((5e-5, 2.0, 10), (0.0, 0.0, 3)):
        print(kind, nbits, alpha, flush=True)
        check(ctx, [draw(n, 31 * n + nbits, kind) for n in SIZES], nbits, iters, alpha, beta)


@pytest.mark.parametrize("flags", [X.EXCP_FLAG_W_F16, X.EXCP_FLAG_W_BF16, X.EXCP_FLAG_NO_M2W])
@pytest.mark.parametrize("kind", ["spread", "tied"])
def test_storages_and_the_scalar_threshold(ctx, kind, flags):
    for nbits in (3, 8):
        check(ctx, [draw(n, n + nbits, kind, flags) for n in SIZES], nbits, 5, 5e-5 if flags != X.EXCP_FLAG_NO_M2W else 0.5, 1.0, flags)


@pytest.mark.parametrize("sign", [1, -1])
def test_zeros_among_the_second_moments(ctx, sign):
    # (kept where the threshold does not depend on them; nothing but zeros in the last)
    cases = []
    for n, zeros in ((100, 1), (4096, 20), (8192, 400), (8192, 8000), (700, 700)):
        Wp, W, m, v = draw(n, n + zeros, "spread")
        v[np.random.default_rng(zeros).choice(n, zeros, replace=False)] = 0.0
        cases.append((Wp, W, m, v if sign > 0 else -v))
    for nbits in (2, 4, 8):
        check(ctx, cases, nbits, 4, 0.0, 0.0, X.EXCP_FLAG_NO_M2W)


@pytest.mark.parametrize("n", [1, 777, 8192, 8193])
def test_alone_and_over_the_previous_weights(ctx, n):
    check(ctx, [draw(n, n, "spread")], 4, 10, in_place=True)
    check(ctx, [draw(n, n, "spread")], 4, 0)


@pytest.mark.parametrize("nbits", [4, 8])           # one wave's centres, and more
@pytest.mark.parametrize("where", ["W_prev", "W_t", "W_prev of one"])
def test_over_their_inputs_beside_tensors_that_fill_the_gpu(where, nbits):
    """W_hat over what a workgroup of the same tensor reads, while larger tensors hold the compute units and workgroups begin far apart: the
    blobs and W_hat are the oracle's, and those of the larger tensors (in place too) what the call that leaves its inputs alone gives."""
    small = [draw(4096 if i % 4 else 8192 - i, 100 * nbits + i, "spread") for i in range(40)]
    g = torch.Generator(device="cuda").manual_seed(nbits)
    large = []
    for n in (18_000_001, 16_777_216, 16_777_216):
        Wp, d, m = (torch.empty(n, device="cuda").normal_(0, s, generator=g) for s in (0.02, 1.4e-4, 5e-5))
        large.append((Wp, Wp + d, m, torch.empty(n, device="cuda").normal_(generator=g).exp_().mul_(m).mul_(m).add_(1e-16)))
    c = X.Context(18_000_001, 60_000_000)
    refs = [O.compress_step(*t, 5e-5, 2.0, nbits, 4) for t in small]
    wants = [O.decompress_step(t[0], r.blob)[0] for t, r in zip(small, refs)]

    def go(over):
        """The call with W_hat in arrays of its own, or over its inputs: blobs and W_hat of all tensors."""
        items = []
        for i, t in enumerate([tuple(torch.from_numpy(a).cuda() for a in t) for t in small] + [tuple(a.clone() for a in t) for t in large]):
            out = torch.zeros_like(t[0])
            if over and (where != "W_prev of one" or i in (20, 41)):
                out = t[1] if where == "W_t" else t[0]
            items.append((*t, torch.zeros(X.excp_blob_bound(t[0].numel(), nbits), dtype=torch.uint8, device="cuda"), out))
        items = items[:13] + items[40:42] + items[13:40] + items[42:]          # (small ones between the large ones)
        c.excp_compress_tensors(items, 5e-5, 2.0, nbits, 4)
        rc, stats = c.excp_collect(check=False)
        assert rc == 0
        at = list(range(13)) + list(range(15, 42)) + [13, 14, 42]              # the order they were made in
        return [(items[i][4][:stats[i].blob_bytes], items[i][5], stats[i]) for i in at]

    apart, over = go(False), go(True)
    for got in (apart, over):
        for (blob, out, st), ref, want in zip(got, refs, wants):
            assert (st.n_w, st.n_o) == (ref.n_w, ref.n_o) and blob.cpu().numpy().tobytes() == ref.blob
            assert out.cpu().numpy().tobytes() == want.tobytes()
    for a, b in zip(apart[40:], over[40:]):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1].view(torch.int32), b[1].view(torch.int32))
    c.close()


def test_small_tensors_beside_a_larger_one(ctx):
    """The larger one takes the general kernels, the others their own on the context's second stream: timed there, in one span."""
    cases = [draw(n, n, "spread") for n in (100, 8192, 8193)]
    check(ctx, cases, 4, 10)
    ctx.excp_set_profiling(True)
    try:
        for part, spans in ((cases, (1, 1, 1)), (cases[:2], (1, 1, 0)), (cases[2:], (1, 0, 1))):
            check(ctx, part, 4, 10)
            t = ctx.stage_times()
            assert (t["layout"][1], t["misc"][1], t["mask_slots"][1]) == spans
            assert t["misc"][0] > 0 or not spans[1]
    finally:
        ctx.excp_set_profiling(False)


@pytest.mark.parametrize("nbits", [4, 8])
def test_several_groups_of_small_and_larger_tensors(nbits):
    """Groups follow one another through the same areas while small tensors go beside the larger ones: with larger tensors whose
    Lloyd iterations may be shared out (they join the second stream themselves), without any such, and alone."""
    r = np.random.default_rng(nbits)
    sizes = [300_000, 8192, 100, 90_000, 5000, 8193, 8000, 20_000, 300_001, 1, 700, 60_000, 3000, 64, 8191, 30_000, 9000, 4096, 40_001, 2000]
    cases = [draw(n, int(r.integers(1 << 30)), ("spread", "tied", "crowded")[i % 3]) for i, n in enumerate(sizes)]
    c = X.Context(300_001, 310_000)
    c.excp_set_profiling(True)
    try:
        for _ in range(3):
            check(c, cases, nbits, 3, in_place=True)
            t = c.stage_times()
            assert t["layout"][1] >= 3 and t["misc"][1] >= 3
    finally:
        c.close()


def test_errors_stay_with_their_tensor(ctx):
    cases = [draw(500, i, "spread") for i in range(4)]
    cases[1][3][7] = np.inf
    cases[2][1][9] = np.nan
    rc, stats, items, outs = run(ctx, cases, 4, 5, 5e-5, 2.0, 0)
    assert rc == X.EXCP_E_NONFINITE
    assert [s.status for s in stats] == [0, X.EXCP_E_NONFINITE, X.EXCP_E_NONFINITE, 0] and stats[1].nonfinite == 1 and stats[2].nonfinite == 1
    for i in (0, 3):
        assert items[i][4][:stats[i].blob_bytes].cpu().numpy().tobytes() == O.compress_step(*cases[i], 5e-5, 2.0, 4, 5).blob
    assert not outs[1].any() and not outs[2].any()          # nothing is reconstructed from a tensor that failed
    # capacity: exactly enough, and sixteen bytes less
    c = draw(3000, 5, "spread")
    size = len(O.compress_step(*c, 0.0, 0.0, 4, 2).blob)
    for cap, want in ((size, 0), (size - 16, X.EXCP_E_CAP)):
        blob = torch.full((size + 64,), 0xAB, dtype=torch.uint8, device="cuda")
        t = [torch.from_numpy(a).cuda() for a in c]
        ctx.excp_compress_tensors([(*t, blob[:cap], None)], 0.0, 0.0, 4, 2)
        rc, st = ctx.excp_collect(check=False)
        assert rc == want and st[0].blob_bytes == size and (blob[cap:] == 0xAB).all()
