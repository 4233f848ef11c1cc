"""milora_routed_linear where its launches change hands: slices of rows, tenants that share a tile, workspaces that served
other calls.  Host-side answers are checked on the CPU, results on the GPU against the fp64 oracle or fp64 torch."""
import pytest
import torch

import oracle
from paper_2410_18035_amd import binding as mb
from paper_2410_18035_amd import synth
from tests.util import assert_rows_close, oracle_adapters, to_f64

DEV = "cuda:0"
gpu = pytest.mark.gpu


def _adapters(T, d1, d2, ranks, sigma, seed, dtype=torch.bfloat16):
    """Adapter matrices of T tenants for one linear of d1 x d2, the same at all seven sites."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    rnd = lambda *s: torch.empty(*s, dtype=torch.float32, device=DEV).normal_(0, sigma, generator=g).to(dtype)
    rank = [ranks[t % len(ranks)] for t in range(T)]
    A = [[rnd(d1, r)] * 7 for r in rank]
    B = [[rnd(r, d2)] * 7 for r in rank]
    return A, B, rank


@gpu
def test_second_slice_of_unmapped_rows_keeps_its_requests():
    """A row-major weight of 4 GiB is beyond the 256 x 256 kernel's offsets: its rows go in slices of 4096 through the smaller
    tiles.  Without a row map, row m belongs to request m in every slice: the requests behind row 4096 have a tenant of their
    own, those of the same place in the first slice no LoRA term."""
    d1, d2, M = 1 << 18, 1 << 13, 4100
    assert 2 * d1 * d2 >= 1 << 32
    g = torch.Generator(device=DEV).manual_seed(5)
    W = torch.empty(d2, d1, dtype=torch.bfloat16, device=DEV)
    for n in range(0, d2, 512):
        W[n:n + 512] = torch.empty(512, d1, dtype=torch.float32, device=DEV).normal_(0, d1 ** -0.5, generator=g)
    X = torch.empty(M, d1, dtype=torch.float32, device=DEV).normal_(0, 1, generator=g).to(torch.bfloat16)
    A, B, rank = _adapters(3, d1, d2, (8, 16), 0.03, 6)
    tab = mb.AdapterTable.from_tensors(A, B, rank)
    tid = torch.tensor([2 if m >= 4096 else m % 2 for m in range(M)], dtype=torch.int32)
    route = torch.full((M,), 4, dtype=torch.uint8)
    route[:4] = mb.ROUTE_NONE
    Y = mb.milora_routed_linear(X, W, tab, 4, tid.to(DEV), route.to(DEV))
    rows = [0, 1, 4, 5, 4094, 4095, 4096, 4097, 4099]
    x = X[rows].double()
    ref = torch.cat([x @ W[n:n + 512].double().T for n in range(0, d2, 512)], 1)
    for i, m in enumerate(rows):
        if route[m] == 4:
            delta = (x[i] @ A[tid[m]][4].double()) @ B[tid[m]][4].double()
            assert delta.abs().max() > 0.2 * ref[i].abs().max()  # a lost or foreign term shows
            ref[i] += delta
    assert_rows_close(Y[rows], ref.cpu().numpy(), torch.bfloat16)


@gpu
def test_slices_of_mapped_rows_on_packed_weights():
    """Packed rows beyond 4096 go in slices of their own, the last of them ragged."""
    wl = synth.Workload("s", "bf16", 96, 208, 1, 5, 9, (5, 16), (3, 40), tenants="uniform", seed=8, sigma_w=0.05, sigma_lora=0.15)
    W, ad = synth.base_weights(wl, 0, DEV), synth.adapters(wl, 0, DEV)
    tab = mb.AdapterTable.from_tensors(ad.A, ad.B, ad.rank)
    g = torch.Generator().manual_seed(9)
    M, site = 4096 + 33, 5
    X = torch.randn(M, wl.d, generator=g).to(torch.bfloat16).to(DEV)
    r2r = torch.randint(0, wl.B, (M,), generator=g).to(torch.int32)
    tid, route = synth.tenant_ids(wl), torch.tensor([5, 5, 0, 5, 5, 2, 5, 255, 5], dtype=torch.uint8)
    Y = mb.milora_routed_linear(X, mb.milora_pack_weight(W[site]), tab, site, tid.to(DEV), route.to(DEV), r2r.to(DEV),
                                w_layout=mb.W_PACKED, d2=wl.F)
    ref = oracle.routed_linear(synth.as_numpy(X), synth.as_numpy(W[site]), oracle_adapters(ad), site, tid.numpy(), route.numpy(),
                               row_to_req=r2r.numpy())
    assert_rows_close(Y, ref, torch.bfloat16)


def test_workspace_for_the_largest_call_serves_every_smaller_one():
    """A caller sizes its workspace once: no fewer rows, narrower weights or smaller ranks may need more."""
    size = mb.routed_linear_workspace_bytes
    rows = [1, 16, 17, 32, 33, 63, 64, 65, 96, 128, 129, 255, 256, 257, 300, 512, 513, 777, 1024, 1025, 2048, 2049, 4095, 4096,
            4097, 4160, 8192, 8193, 16384, 32768, 32769, 1 << 20]
    widths = [1, 3, 16, 64, 96, 128, 1000, 1024, 1025, 2048, 2049, 4096, 4160, 8193, 11008, 13824, 100_000]
    for r in (1, 5, 8, 64, 256):
        for a in widths:
            for b in widths:
                assert all(x <= y for x, y in zip(*[[size(M, a, b, r) for M in rows][i:] for i in (0, 1)])), (a, b, r)
        for M in (1, 45, 96, 300, 512, 4096, 5000):
            for a in widths:
                along = [size(M, a, b, r) for b in widths], [size(M, b, a, r) for b in widths]
                assert all(x <= y for s in along for x, y in zip(s, s[1:])), (M, a, r)
    for M in rows:
        assert size(M, 4096, 4096, 8) <= size(M, 4096, 4096, 9) <= size(M, 4096, 4096, 64)


@gpu
@pytest.mark.parametrize("packed,M,d1,d2,T", [
    (False, 45, 192, 272, 5),    # 64 x 64 tiles, one part
    (False, 63, 4096, 144, 7),   # the reduction in parts
    (True, 33, 96, 2064, 33),    # a tenant per row, half a stage at the end
    (True, 100, 2048, 3520, 9),  # 128 x 128 tiles
    (False, 130, 192, 272, 6),   # the LoRA term as matrix stages, 64 x 64 tiles
    (False, 300, 2048, 3520, 9),  # 128 x 128 tiles, in parts
    (False, 4097, 192, 272, 40),  # 256 x 256 tiles
])
def test_one_tenants_infinities_and_nans_reach_its_own_rows_only(packed, M, d1, d2, T):
    """Rows of many tenants meet in a tile.  Tenant 1's W^B holds Inf and NaN, tenant 2's W^A an Inf (its shrink is Inf): every
    other row, routed or not, stays bit for bit what it is with clean adapters, and theirs are Inf and NaN where fp64 has them."""
    site, rank = 2, (12, 16, 5)
    A, B, ranks = _adapters(T, d1, d2, rank, 0.1, 30 + M)
    A, B = [[a[0].clone()] * 7 for a in A], [[b[0].clone()] * 7 for b in B]
    g = torch.Generator(device=DEV).manual_seed(M)
    rnd = lambda *s: torch.empty(*s, dtype=torch.float32, device=DEV).normal_(0, 1, generator=g).to(torch.bfloat16)
    X, W = rnd(M, d1), rnd(d2, d1) * d1 ** -0.5
    Wd = mb.milora_pack_weight(W) if packed else W
    tid = torch.arange(T, dtype=torch.int32)
    route = torch.tensor([mb.ROUTE_NONE if t == 4 else site for t in range(T)], dtype=torch.uint8)
    r2r = (torch.arange(M) % T).to(torch.int32)
    run = lambda: mb.milora_routed_linear(X, Wd, mb.AdapterTable.from_tensors(A, B, ranks), site, tid.to(DEV), route.to(DEV),
                                          r2r.to(DEV), w_layout=mb.W_PACKED if packed else mb.W_ROWMAJOR, d2=d2)
    clean = run()
    assert torch.isfinite(clean).all()
    for c, n, v in [(3, 7, float("inf")), (0, d2 - 1, float("-inf")), (ranks[1] - 1, 64, float("nan"))]:
        B[1][site][c, n] = v
    A[2][site][d1 - 1, 1] = float("inf")
    Y = run()
    bad = (r2r == 1) | (r2r == 2)
    assert torch.equal(Y[~bad], clean[~bad])
    for m in torch.nonzero(bad).flatten().tolist()[:60]:
        t = X[m].double() @ A[r2r[m]][site].double()
        ref = X[m].double() @ W.double().T + (t[:, None] * B[r2r[m]][site].double()).sum(0)
        # (as the sum of two bf16 values, an infinite t is Inf and Inf - Inf)
        split = not packed and M >= 64 and not torch.isfinite(t).all()
        for kind in (lambda v: ~torch.isfinite(v),) if split else (torch.isnan, torch.isposinf, torch.isneginf):
            assert torch.equal(kind(Y[m]), kind(ref)), f"row {m}, tenant {int(r2r[m])}"
        fine = torch.isfinite(ref)
        if fine.any():
            assert (Y[m].double() - ref)[fine].abs().max() <= 2e-2 * ref[fine].abs().max()


@gpu
@pytest.mark.parametrize("packed,M", [(False, 1), (False, 63), (True, 1), (True, 33), (True, 200)])
def test_the_low_rank_intermediate_keeps_all_bits(packed, M):
    """t = 2^20 + 2^10 + 1, every sum exact in fp32, against a base term of -(2^20 + 2^10): the result is the last of t's 21 bits."""
    d1, d2, site = 64, 80, 0
    X, W = torch.zeros(M, d1), torch.zeros(d2, d1)
    X[:, 5], X[:, 20], X[:, 63] = 2.0 ** 10, 2.0 ** 5, 1.0
    W[:, 5], W[:, 20] = -2.0 ** 10, -2.0 ** 5
    A, B = torch.zeros(d1, 8), torch.zeros(8, d2)
    A[5, 3], A[20, 3], A[63, 3], B[3] = 2.0 ** 10, 2.0 ** 5, 1.0, 1.0
    X, W, A, B = (v.to(torch.bfloat16).to(DEV) for v in (X, W, A, B))
    tab = mb.AdapterTable.from_tensors([[A] * 7], [[B] * 7], [8])
    one = torch.zeros(1, dtype=torch.uint8, device=DEV)
    Y = mb.milora_routed_linear(X, mb.milora_pack_weight(W) if packed else W, tab, site, one.int(), one,
                                torch.zeros(M, dtype=torch.int32, device=DEV), w_layout=mb.W_PACKED if packed else mb.W_ROWMAJOR, d2=d2)
    assert (Y == 1).all()


@gpu
@pytest.mark.parametrize("packed,M,d1,d2", [
    (False, 16, 4096, 64),    # few rows, the reduction in parts
    (False, 300, 2048, 3520),  # 128 x 128 tiles in parts, the LoRA term as matrix stages
    (False, 40, 130, 70),     # any-shape
    (True, 70, 4096, 64),     # packed, in parts
    (True, 4100, 1024, 64),   # packed, a second slice of few rows
])
def test_tiles_work_whatever_the_workspace_holds(packed, M, d1, d2):
    """Parts of a reduction count themselves in words of the workspace: these start from zero in every call."""
    A, B, rank = _adapters(4, d1, d2, (8, 20), 0.1, 50)
    tab = mb.AdapterTable.from_tensors(A, B, rank)
    g = torch.Generator(device=DEV).manual_seed(51)
    rnd = lambda *s: torch.empty(*s, dtype=torch.float32, device=DEV).normal_(0, 1, generator=g).to(torch.bfloat16)
    X, W = rnd(M, d1), rnd(d2, d1)
    W = mb.milora_pack_weight(W) if packed else W
    ids = torch.arange(4, dtype=torch.int32, device=DEV)
    r2r = torch.arange(M, dtype=torch.int32, device=DEV) * 4 // M
    nbytes = mb.routed_linear_workspace_bytes(M, d1, d2, tab.r_max)
    run = lambda ws: mb.milora_routed_linear(X, W, tab, 1, ids, torch.ones_like(ids, dtype=torch.uint8), r2r, d2=d2,
                                             w_layout=mb.W_PACKED if packed else mb.W_ROWMAJOR, workspace=ws,
                                             out=torch.full((M, d2), 7.0, dtype=torch.bfloat16, device=DEV))
    clean = run(torch.zeros(nbytes, dtype=torch.uint8, device=DEV))
    dirty = torch.full((nbytes,), 255, dtype=torch.uint8, device=DEV)
    for _ in range(2):
        assert torch.equal(run(dirty), clean)
    assert torch.equal(run(torch.randint(0, 256, (nbytes,), dtype=torch.uint8, device=DEV)), clean)


@gpu
@pytest.mark.parametrize("M", [1, 17])
def test_any_shape_linears_wider_than_one_launch(M):
    """A grid holds fewer than 2^32 threads: beyond 2^26 columns (of 16 each 512 threads) the launch is cut."""
    d1, d2 = 1, (1 << 27) + 24
    g = torch.Generator(device=DEV).manual_seed(61)
    W = torch.empty(d2, d1, dtype=torch.bfloat16, device=DEV).normal_(0, 1, generator=g)
    X = torch.empty(M, d1, dtype=torch.bfloat16, device=DEV).normal_(0, 1, generator=g)
    A, B, rank = _adapters(1, d1, d2, (1,), 1.0, 62)
    one = torch.zeros(1, dtype=torch.uint8, device=DEV)
    Y = mb.milora_routed_linear(X, W, mb.AdapterTable.from_tensors(A, B, rank), 0, one.int(), one,
                                torch.zeros(M, dtype=torch.int32, device=DEV))
    for n in (0, (1 << 26) - 40, (1 << 27) - 40):
        cols = slice(n, min(n + 80, d2))
        ref = X.double() @ W[cols].double().T + (X.double() @ A[0][0].double()) @ B[0][0][:, cols].double()
        assert (Y[:, cols].double() - ref).abs().max() <= 2e-2 * ref.abs().max()


@gpu
def test_slices_of_unmapped_packed_rows_keep_their_requests():
    """A reduction of 2^23 is beyond the tiles' offsets: packed rows above 32 go through the stream kernel in slices."""
    d1, d2, M, r = 1 << 23, 16, 36, 8
    g = torch.Generator(device=DEV).manual_seed(71)
    rnd = lambda *s, sigma=1.0: torch.empty(*s, dtype=torch.bfloat16, device=DEV).normal_(0, sigma, generator=g)
    W, X = rnd(d2, d1, sigma=d1 ** -0.5), rnd(M, d1)
    A, B, rank = _adapters(2, d1, d2, (r,), 0.02, 72)
    tid = torch.tensor([1 if m >= 32 else 0 for m in range(M)], dtype=torch.int32)
    route = torch.zeros(M, dtype=torch.uint8)
    route[:2] = mb.ROUTE_NONE
    ws = torch.zeros(mb.routed_linear_workspace_bytes(M, d1, d2, r), dtype=torch.uint8, device=DEV)
    Y = mb.milora_routed_linear(X, mb.milora_pack_weight(W), mb.AdapterTable.from_tensors(A, B, rank), 0, tid.to(DEV),
                                route.to(DEV), w_layout=mb.W_PACKED, d2=d2, workspace=ws)
    assert mb.milora_packed_workspace_status(ws) == 0
    rows = [0, 1, 2, 31, 32, 33, 35]
    for m in rows:
        x = X[m].double()
        ref = torch.stack([x @ W[n].double() for n in range(d2)])
        if route[m] == 0:
            delta = torch.stack([x @ A[tid[m]][0][:, c].double() for c in range(r)]) @ B[tid[m]][0].double()
            assert delta.abs().max() > 0.2 * ref.abs().max()
            ref = ref + delta
        assert_rows_close(Y[m:m + 1], ref[None].cpu().numpy(), torch.bfloat16, f"row {m}")


def test_tile_query_follows_the_dispatch():
    """Which matrix-core tiles a call runs on, at the borders of the rules."""
    k, bf, f32 = mb.milora_routed_linear_tile, torch.bfloat16, torch.float32
    assert [k(M, 4096, 4096, bf, mb.W_PACKED) for M in (1, 32, 33)] == [0, 0, 64]
    assert k(96, 4096, 11008, bf, mb.W_PACKED) == 128 and k(32768, 4096, 11008, bf, mb.W_PACKED) == 128
    assert [k(M, 64, 16, bf) for M in (1, 63, 64, 4096, 4097)] == [64, 64, 64, 64, 256]
    assert k(777, 4096, 4096, bf) == 128 and k(777, 4096, 11008, bf) == 256 and k(32768, 4096, 4096, bf) == 256
    assert k(700, 96, 528, bf) == 0 and k(700, 192, 520, bf) == 0 and k(700, 192, 528, f32) == 0
    assert k(5000, 1 << 18, 1 << 13, bf) in (64, 128)  # a weight of 4 GiB: beyond the 256 x 256 kernel's offsets
    assert k(40, 1 << 23, 16, bf, mb.W_PACKED) == 0 and k(40, 1 << 23, 16, bf) == 0  # beyond the smaller tiles' offsets
    assert k(4096, 64, 1 << 23, bf) == 256  # more smaller tiles than a grid of fewer than 2^32 threads holds
    assert k(32, 4096, 4096, f32, mb.W_PACKED) == -3 and k(0, 8, 8, f32) == -1 and k(8, 8, 8, f32, 5) == -1


@gpu
@pytest.mark.parametrize("M,d1,d2,ranks,T,spread", [
    (4097, 64, 272, (5, 40), 7, "segments"),     # one row in the last row tile, a second block of 32 ranks, ranks of any size
    (4400, 192, 528, (16, 64, 33), 5, "segments"),  # a ragged last row tile, three column tiles, a ragged one, r_max % 4 == 0
    (4400, 128, 352, (8, 24), 20, "scattered"),  # tenants of neighbouring rows differ
    (4300, 64, 48, (256, 3), 3, "segments"),     # the largest rank, eight blocks of 32, one narrow column tile
    (8193, 320, 272, (7,), 2, "none"),           # unmapped rows, r_max % 4 != 0
])
def test_routed_linear_256_tiles(M, d1, d2, ranks, T, spread):
    """The 256 x 256 kernel and the 64-row shrink blocks in front of it, with bias, against the fp64 oracle."""
    assert mb.milora_routed_linear_tile(M, d1, d2, torch.bfloat16) == 256
    g = torch.Generator().manual_seed(M + d1)
    rnd = lambda *s, sigma: (torch.randn(*s, generator=g) * sigma).to(torch.bfloat16).to(DEV)
    X, W, bias = rnd(M, d1, sigma=1.0), rnd(d2, d1, sigma=d1 ** -0.5), rnd(d2, sigma=0.1)
    A, B, rank = _adapters(T, d1, d2, ranks, 0.12, M)
    site, nreq = 4, M if spread == "none" else T + 2
    tid = torch.arange(nreq, dtype=torch.int32) % T
    route = torch.randint(0, 7, (nreq,), generator=g).to(torch.uint8)
    route[::2] = site
    r2r = {"segments": torch.sort(torch.randint(0, nreq, (M,), generator=g))[0], "none": None,
           "scattered": torch.randint(0, nreq, (M,), generator=g)}[spread]
    r2r = None if r2r is None else r2r.to(torch.int32)
    Y = mb.milora_routed_linear(X, W, mb.AdapterTable.from_tensors(A, B, rank), site, tid.to(DEV), route.to(DEV),
                                None if r2r is None else r2r.to(DEV), bias=bias)
    ref = oracle.routed_linear(synth.as_numpy(X), synth.as_numpy(W), oracle.Adapters(
        [[synth.as_numpy(a) for a in row] for row in A], [[synth.as_numpy(b) for b in row] for row in B], rank), site, tid.numpy(),
        route.numpy(), row_to_req=None if r2r is None else r2r.numpy(), bias=synth.as_numpy(bias))
    assert_rows_close(Y, ref, torch.bfloat16)


@gpu
@pytest.mark.parametrize("side,M,d1,d2", [(64, 130, 192, 272), (128, 300, 2048, 3520), (256, 4097, 64, 272), (256, 4400, 192, 528)])
def test_tiles_at_the_least_alignment(side, M, d1, d2):
    """W^B and the bias at odd elements, Y eight bytes past a sixteenth: the bits of the aligned call, and nothing written around Y."""
    assert mb.milora_routed_linear_tile(M, d1, d2, torch.bfloat16) == side
    T, site = 5, 3
    A, B, rank = _adapters(T, d1, d2, (16, 33, 64), 0.1, M)
    g = torch.Generator(device=DEV).manual_seed(M + 1)
    rnd = lambda *s: torch.empty(*s, dtype=torch.float32, device=DEV).normal_(0, 1, generator=g).to(torch.bfloat16)
    X, W, bias = rnd(M, d1), rnd(d2, d1) * d1 ** -0.5, rnd(d2)
    tid, route = torch.arange(T, dtype=torch.int32, device=DEV), torch.full((T,), site, dtype=torch.uint8, device=DEV)
    r2r = (torch.arange(M, device=DEV) * T // M).to(torch.int32)
    call = lambda B, bias, Y: mb.milora_routed_linear(X, W, mb.AdapterTable.from_tensors(A, B, rank), site, tid, route, r2r, bias=bias, out=Y)
    aligned = torch.empty(M, d2, dtype=torch.bfloat16, device=DEV)
    assert aligned.data_ptr() % 16 == 0 and all(b[0].data_ptr() % 16 == 0 for b in B)
    call(B, bias, aligned)
    past = lambda t: torch.empty(t.numel() + 1, dtype=t.dtype, device=DEV)[1:].view_as(t).copy_(t)
    around = torch.full((4 + M * d2 + 64,), -7.0, dtype=torch.bfloat16, device=DEV)
    Y = around[4:4 + M * d2].view(M, d2)
    B1, bias1 = [[past(b[0])] * 7 for b in B], past(bias)
    assert Y.data_ptr() % 16 == 8 and bias1.data_ptr() % 4 == 2 and all(b[0].data_ptr() % 4 == 2 for b in B1)
    call(B1, bias1, Y)
    assert torch.equal(Y.view(torch.int16), aligned.view(torch.int16))
    assert (around[:4] == -7).all() and (around[4 + M * d2:] == -7).all()


def test_tile_choice_where_one_is_clearly_faster():
    """Sizes at which one kind of tile takes at least 8 % less time than the next, with every row routed and with none."""
    k = lambda *s: mb.milora_routed_linear_tile(*s, torch.bfloat16)
    assert [k(*s) for s in ((1805, 192, 7488), (600, 5120, 13824), (777, 4096, 11008))] == [256] * 3
    assert [k(*s) for s in ((2048, 4096, 4096), (3846, 512, 1040))] == [128] * 2
    assert k(300, 4096, 11008) != 256


@gpu
@pytest.mark.parametrize("M,d1,d2", [(517, 64, 13312), (517, 64, 13328)])
def test_routed_linear_256_tiles_of_fewer_rows(M, d1, d2):
    """Sizes that both kernels take, the 256 x 256 one by a quarter of the time: a ragged last row tile, whole and ragged columns."""
    test_routed_linear_256_tiles(M, d1, d2, (16, 40), 6, "segments")


@gpu
def test_routed_linear_256_tiles_small_integers_bit_exact():
    d1, d2, T, r, M, site = 64, 272, 3, 4, 4200, 1
    rnd = lambda shape, lo, hi, seed: synth.small_int_tensor(shape, lo, hi, torch.bfloat16, seed, DEV)
    assert mb.milora_routed_linear_tile(M, d1, d2, torch.bfloat16) == 256
    X, W = rnd((M, d1), -2, 2, 2), rnd((d2, d1), -1, 1, 1)
    A, B = [[rnd((d1, r), -1, 1, 300 + t)] * 7 for t in range(T)], [[rnd((r, d2), -1, 1, 400 + t)] * 7 for t in range(T)]
    tid = torch.tensor([0, 1, 2, 2, 1, 0], dtype=torch.int32)
    route = torch.tensor([site, 0, site, site, 3, site], dtype=torch.uint8)
    r2r = (torch.arange(M) * 6 // M).to(torch.int32)
    Y = mb.milora_routed_linear(X, W, mb.AdapterTable.from_tensors(A, B, [r] * T), site, tid.to(DEV), route.to(DEV), r2r.to(DEV))
    ref = oracle.routed_linear(synth.as_numpy(X), synth.as_numpy(W), oracle.Adapters(
        [[synth.as_numpy(a) for a in row] for row in A], [[synth.as_numpy(b) for b in row] for row in B], [r] * T), site,
        tid.numpy(), route.numpy(), row_to_req=r2r.numpy())
    assert (abs(ref) <= 256).all()
    assert (to_f64(Y) == ref).all()


@gpu
@pytest.mark.parametrize("packed,M,d1,d2", [(False, 16, 4096, 64), (False, 300, 2048, 3520), (True, 70, 4096, 64)])
def test_tiles_in_parts_replay_in_a_graph(packed, M, d1, d2):
    """Shrink, counters and parts recorded once and replayed on new rows, with eager calls on the same workspace between."""
    A, B, rank = _adapters(4, d1, d2, (8, 20), 0.1, 80)
    tab = mb.AdapterTable.from_tensors(A, B, rank)
    g = torch.Generator(device=DEV).manual_seed(81)
    rnd = lambda *s: torch.empty(*s, dtype=torch.float32, device=DEV).normal_(0, 1, generator=g).to(torch.bfloat16)
    X, W = rnd(M, d1), rnd(d2, d1)
    W = mb.milora_pack_weight(W) if packed else W
    ids = torch.arange(4, dtype=torch.int32, device=DEV)
    r2r, route = torch.arange(M, dtype=torch.int32, device=DEV) * 4 // M, torch.ones(4, dtype=torch.uint8, device=DEV)
    ws = torch.zeros(mb.routed_linear_workspace_bytes(M, d1, d2, tab.r_max), dtype=torch.uint8, device=DEV)
    out = torch.empty(M, d2, dtype=torch.bfloat16, device=DEV)
    run = lambda x, y: mb.milora_routed_linear(x, W, tab, 1, ids, route, r2r, d2=d2, w_layout=mb.W_PACKED if packed else mb.W_ROWMAJOR,
                                               workspace=ws, out=y)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run(X, out)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(X, out)
    for rep in range(5):
        x = rnd(M, d1)
        eager = run(x, torch.empty_like(out)).clone()
        torch.cuda.synchronize()
        X.copy_(x)
        out.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager), f"replay {rep}"
