"""Scans that leave maxima, and the selection from them, at the edges of their
tiles (GPU).

Embeddings are small integers, so every product, sum and distance is exact in
fp32 and bf16 and many rows are equally far: the reference is an integer
computation sorted by (distance, index), and the neighbours must match it
exactly, ties included.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"


def draw(B, N, d, dtype, lo, hi, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    bank = torch.randint(lo, hi + 1, (N, d), generator=g, device=DEV).to(t)
    q = torch.randint(lo, hi + 1, (B, d), generator=g, device=DEV).to(t)
    return q, bank


def reference(q, bank, k):
    """(index, distance) of the k first rows by (distance, index); chunks of the
    bank in float64 (exact for these integers)."""
    q = q.double()
    keys = []
    for r0 in range(0, bank.shape[0], 1 << 18):
        x = bank[r0:r0 + (1 << 18)].double()
        dist = (q * q).sum(1)[:, None] + (x * x).sum(1)[None] - 2 * (q @ x.t().contiguous())
        key = dist * float(1 << 32) + torch.arange(r0, r0 + x.shape[0], device=DEV)
        keys.append(torch.topk(key, min(k, x.shape[0]), dim=1, largest=False).values)
    key = torch.topk(torch.cat(keys, 1), k, dim=1, largest=False).values.sort(dim=1).values
    dist = torch.floor(key / float(1 << 32))
    return (key - dist * float(1 << 32)).to(torch.int32), dist.float()


def check(q, bank, k, label):
    import paper_2606_17949_amd as rb
    print(label, flush=True)
    idx, dist = rb.rb_knn_topk(q, bank, rb.rb_bank_norms(bank), k)
    torch.cuda.synchronize()
    ref_idx, ref_dist = reference(q, bank, k)
    assert torch.equal(dist, ref_dist), label
    assert torch.equal(idx, ref_idx), label


@pytest.mark.parametrize("dtype,B,N,d,k", [
    ("f32", 1, 1, 4, 1),              # one row, one k-step, one lane group
    ("f32", 1, 17, 8, 17),            # fewer super tiles than neighbours
    ("f32", 17, 2_047, 20, 10),       # second request group nearly empty, ragged row
    ("f32", 100, 5_003, 300, 20),     # seven groups, rows of 18.75 k-steps
    ("f32", 130, 40_001, 12, 64),     # two request tiles, k at its maximum
    ("f32", 33, 300_017, 16, 10),     # super tiles of two row tiles, the last partial
    ("f32", 5, 1_000_003, 8, 10),     # super tiles of four row tiles
    ("f32", 20, 1_200_007, 8, 20),    # ... of eight
    ("bf16", 64, 2_200_021, 8, 10),   # ... of sixteen
    ("f32", 300, 150_003, 512, 10),   # more super tiles to a wave than it holds
    ("f32", 3, 70, 2_048, 5),         # the longest rows
    ("f32", 92, 9_001, 1_024, 10),    # three request tiles of 85 chunks, five of them spread out
    ("f32", 640, 3_001, 2_048, 4),    # forty request tiles, fewer chunks than XCDs
    ("bf16", 1, 1_000, 8, 10),
    ("bf16", 64, 100_003, 64, 10),
    ("bf16", 49, 33_333, 1_000, 7),   # ragged bf16 rows, four groups
    ("bf16", 64, 4_100, 1_536, 10),   # two request tiles of two groups
])
def test_neighbours_are_exact(dtype, B, N, d, k):
    q, bank = draw(B, N, d, dtype, -2, 2, 1)
    check(q, bank, k, f"exact {dtype} B={B} N={N} d={d} k={k}")


@pytest.mark.parametrize("dtype,B,d", [("f32", 5, 16), ("bf16", 5, 64)])
def test_equal_rows_come_in_index_order(dtype, B, d):
    """Every row equal: more equal super tiles than the selection holds, and
    the first k rows win."""
    q, bank = draw(B, 40_000, d, dtype, -2, 2, 2)
    bank[:] = bank[0]
    check(q, bank, 10, f"equal rows {dtype}")
    bank[39_000] = q[0]   # and one nearer row
    check(q, bank, 64, f"equal rows but one {dtype}")


@pytest.mark.parametrize("dtype,B,N,d,k", [
    ("f32", 33, 40_000, 16, 10),       # single row tiles
    ("f32", 9, 300_017, 16, 10),       # super tiles of two
    ("bf16", 64, 2_200_021, 8, 20),    # ... of sixteen
    ("bf16", 200, 33_000, 768, 10),    # query-resident
    ("bf16", 100, 150_001, 768, 64),
    ("bf16", 300, 33_000, 768, 10),    # GEMM-structured, half-size workgroups
    ("bf16", 150, 40_003, 136, 33),
])
def test_banks_in_the_order_of_their_clusters(dtype, B, N, d, k):
    """Near rows that follow one another: most row tiles of the k super tiles
    are near, and the super tiles are one another's neighbours."""
    q, bank = draw(B, N, d, dtype, -1, 1, 10)
    g = torch.Generator(device=DEV).manual_seed(11)
    n_c = max(4, N // 2_500)
    centre = torch.randint(-2, 3, (n_c, d), generator=g, device=DEV).to(bank.dtype)
    bank += centre[torch.arange(N, device=DEV) * n_c // N]
    q += centre[torch.randint(0, n_c, (B,), generator=g, device=DEV)]
    check(q, bank, k, f"clusters in order {dtype} B={B} N={N} d={d} k={k}")


def test_rows_that_are_no_numbers_are_no_neighbours():
    """Fewer rows with a distance than neighbours: index -1, distance NaN."""
    import paper_2606_17949_amd as rb
    q, bank = draw(2, 40, 16, "f32", -2, 2, 3)
    norms = rb.rb_bank_norms(bank)
    norms[7:] = float("nan")
    print("rows without a distance", flush=True)
    idx, dist = rb.rb_knn_topk(q, bank, norms, 10)
    torch.cuda.synchronize()
    assert torch.all(idx[:, 7:] == -1) and torch.all(torch.isnan(dist[:, 7:]))
    assert torch.equal(idx[:, :7].sort(1).values.cpu(),
                       torch.arange(7, dtype=torch.int32).repeat(2, 1))


def test_bank_in_parts_matches_one_pass():
    """The no-allocation call holds the maxima of 64 MiB; a longer bank goes by
    in parts whose neighbours are merged, with the results of one pass."""
    import paper_2606_17949_amd as rb
    B, N, d, k, M, I = 64, 4_200_005, 8, 10, 2, 3
    q, bank = draw(B, N, d, "f32", -3, 3, 4)
    norms = rb.rb_bank_norms(bank)
    g = torch.Generator(device=DEV).manual_seed(5)
    qual = torch.rand(N, M, generator=g, device=DEV)
    length = 100.0 + qual
    plen = torch.full((B,), 50, dtype=torch.int32, device=DEV)
    out = []
    for fn in (rb.rb_route_batch, rb.rb_route_batch_noalloc):
        inst = rb.DeviceInstances(torch.tensor([0, 1, 1], dtype=torch.int32, device=DEV),
                                  *[torch.ones(I, device=DEV) for _ in range(6)])
        r = dict(assign=torch.empty(B, dtype=torch.int32, device=DEV),
                 nbr_idx=torch.empty(B, k, dtype=torch.int32, device=DEV),
                 nbr_dist=torch.empty(B, k, device=DEV), q_hat=torch.empty(B, M, device=DEV),
                 l_hat=torch.empty(B, M, device=DEV))
        print("bank in parts", fn.__name__, flush=True)
        fn(q, bank, norms, k, qual, length, plen, inst, (0.4, 0.3, 0.3), **r)
        torch.cuda.synchronize()
        out.append(r)
    for f in out[0]:
        assert torch.equal(out[0][f], out[1][f]), f
    ref_idx, ref_dist = reference(q, bank, k)
    assert torch.equal(out[0]["nbr_idx"], ref_idx) and torch.equal(out[0]["nbr_dist"], ref_dist)


@pytest.mark.parametrize("B,N,parts", [
    (256, 1_000_003, 1),        # folded entries, one part
    (512, 1_700_013, 2),        # two parts of folded entries, the last one shorter
])
def test_bank_in_parts_query_resident(B, N, parts):
    """The no-allocation call over banks whose maxima would not fit its array:
    the results of one pass, and the integer neighbours of some requests."""
    import paper_2606_17949_amd as rb
    d, k, M, I = 384, 10, 2, 3
    q, bank = draw(B, N, d, "bf16", -1, 1, 12)
    # exact ties across the parts
    bank[N - 40:] = bank[:40]
    q[:20] = bank[:20]
    norms = rb.rb_bank_norms(bank)
    g = torch.Generator(device=DEV).manual_seed(13)
    qual = torch.rand(N, M, generator=g, device=DEV)
    length = 100.0 + qual
    plen = torch.full((B,), 50, dtype=torch.int32, device=DEV)
    out = []
    for fn in (rb.rb_route_batch, rb.rb_route_batch_noalloc):
        inst = rb.DeviceInstances(torch.tensor([0, 1, 1], dtype=torch.int32, device=DEV),
                                  *[torch.ones(I, device=DEV) for _ in range(6)])
        r = dict(assign=torch.empty(B, dtype=torch.int32, device=DEV),
                 nbr_idx=torch.empty(B, k, dtype=torch.int32, device=DEV),
                 nbr_dist=torch.empty(B, k, device=DEV), q_hat=torch.empty(B, M, device=DEV),
                 l_hat=torch.empty(B, M, device=DEV))
        print(f"query-resident, {parts} parts, B={B} N={N}", fn.__name__, flush=True)
        fn(q, bank, norms, k, qual, length, plen, inst, (0.4, 0.3, 0.3), **r)
        torch.cuda.synchronize()
        out.append(r)
    for f in out[0]:
        assert torch.equal(out[0][f], out[1][f]), f
    some = torch.arange(0, B, B // 32, device=DEV)
    ref_idx, ref_dist = reference(q[some], bank, k)
    assert torch.equal(out[0]["nbr_idx"][some], ref_idx)
    assert torch.equal(out[0]["nbr_dist"][some], ref_dist)


@pytest.mark.parametrize("B,N,k", [
    (1_024, 4_300_013, 10),     # folded entries, one part
    (4_096, 3_500_017, 20),     # two parts of them
])
def test_bank_in_parts_gemm(B, N, k):
    """More than 1 GiB of maxima after the GEMM-structured scan: the integer
    neighbours of some requests of every request tile."""
    import paper_2606_17949_amd as rb
    q, bank = draw(B, N, 8, "bf16", -3, 3, 14)
    need = rb.rb_workspace_size(B, N, 8, rb.RB_BF16, k, 1)
    print(f"GEMM-structured, parts, B={B} N={N}: workspace {need / 2**20:.0f} MiB", flush=True)
    assert need < B * (N // 256) * 68
    idx, dist = rb.rb_knn_topk(q, bank, rb.rb_bank_norms(bank), k)
    torch.cuda.synchronize()
    some = torch.arange(5, B, B // 32, device=DEV)
    ref_idx, ref_dist = reference(q[some], bank, k)
    assert torch.equal(dist[some], ref_dist)
    assert torch.equal(idx[some], ref_idx)


@pytest.mark.parametrize("B,N,d,k", [
    (65, 4_099, 384, 64),       # query-resident, one group per wave, last chunk of 3 rows
    (130, 70_001, 384, 10),     # two groups, row halves
    (250, 33_000, 384, 10),     # four groups, row halves
    (512, 66_007, 384, 10),     # four groups, tiles one after the other
    (64, 600_011, 512, 10),     # a small batch over a long bank
    (200, 50_021, 512, 33),
    (256, 20_011, 768, 10),
    (100, 9_000, 768, 1),
    (128, 30_007, 1_024, 10),
    (65, 5_000, 1_024, 10),
    (129, 4_001, 1_024, 10),    # GEMM-structured: one request past the query-resident scan
    (300, 20_003, 768, 20),     # second request tile nearly empty
    (600, 10_000, 384, 10),
    (70, 777, 8, 10),           # one 16-byte piece of a row: a stage of padding
    (128, 5_000, 200, 64),      # tiles of 128 requests, ragged rows
    (90, 3_000, 1_000, 10),
    (1_025, 2_050, 136, 10),    # nine request tiles, every value kept
    (1_025, 9_000, 136, 10),    # five request tiles
    (257, 8_192, 640, 8),       # values kept at the fewest requests, most rows
    (257, 8_193, 640, 8),       # ... and one row more
    (700, 1_025, 768, 1),       # one neighbour, one row past what it keeps
    (300, 2_000, 768, 64),
    (400, 8_192, 1_032, 10),    # too long for that: the GEMM-structured scan, values kept
    (129, 15_360, 1_024, 10),   # values kept over the longest bank of these rows
    (129, 15_361, 1_024, 10),   # ... and one row more
    (70, 777, 640, 64),         # 128 requests a tile, values kept, chunks of 16 rows
    (1_025, 40_011, 1_000, 33), # chunks of several macro tiles, the last one short
    (64, 70_001, 1_536, 10),    # a small batch too long for LDS as one tile
    (33, 65_536, 2_048, 10),    # ... at the fewest requests and rows
    (33, 65_535, 2_048, 10),    # ... and one row below
    (1_151, 11_013, 384, 64),   # fewer super tiles than neighbours: many rounds of rows
    (1_025, 700, 136, 64),      # ... one round
    (1_030, 1_100, 1_000, 40),  # ... a short second one
])
def test_bf16_scans_are_exact(B, N, d, k):
    q, bank = draw(B, N, d, "bf16", -1, 1, 6)
    check(q, bank, k, f"exact bf16 B={B} N={N} d={d} k={k}")


@pytest.mark.parametrize("B,d", [(200, 768), (300, 768), (100, 136)])
def test_bf16_equal_rows_come_in_index_order(B, d):
    q, bank = draw(B, 33_000, d, "bf16", -1, 1, 7)
    bank[:] = bank[5]
    bank[12_345] = q[0]
    check(q, bank, 20, f"equal rows bf16 B={B} d={d}")


@pytest.mark.parametrize("dtype,B,N,d", [
    ("f32", 3, 40, 16),          # every row's value kept
    ("f32", 33, 40_000, 16),     # row tiles computed again
    ("bf16", 5, 9_000, 1_000),
    ("bf16", 100, 9_000, 768),   # query-resident
    ("bf16", 300, 9_000, 768),   # GEMM-structured
])
def test_infinite_distances(dtype, B, N, d):
    """Rows whose norm overflows are at an infinite distance, after all others
    and in index order; an infinite request is at no distance from any row:
    index -1, distance NaN."""
    import paper_2606_17949_amd as rb
    q, bank = draw(B, N, d, dtype, 1, 2, 8)
    near = torch.arange(7, device=DEV) * (N // 7) + N // 14
    far = torch.ones(N, dtype=torch.bool, device=DEV)
    far[near] = False
    bank[far] *= 1e20
    bank[:, d - 1] *= -1
    q[1, d // 2] = float("inf")       # all products +inf
    q[0, d - 1] = float("inf")        # all products -inf
    label = f"infinite distances {dtype} B={B} N={N} d={d}"
    print(label, flush=True)
    idx, dist = rb.rb_knn_topk(q, bank, rb.rb_bank_norms(bank), 10)
    torch.cuda.synchronize()
    assert torch.all(idx[:2] == -1) and torch.all(torch.isnan(dist[:2])), label
    idx, dist = idx[2:], dist[2:]
    assert torch.equal(idx[:, :7].sort(1).values, near.to(torch.int32).expand(B - 2, 7)), label
    assert torch.all(torch.isfinite(dist[:, :7])), label
    ref = torch.nonzero(far)[:3, 0].to(torch.int32)
    assert torch.equal(idx[:, 7:], ref.expand(B - 2, 3)), label
    assert torch.all(dist[:, 7:] == float("inf")), label


@pytest.mark.parametrize("dtype,B,N,d,k", [
    ("f32", 33, 20_000, 300, 10),
    ("bf16", 40, 40_000, 1_000, 10),
    ("bf16", 100, 20_000, 768, 20),     # query-resident
    ("bf16", 300, 20_000, 768, 10),     # GEMM-structured
    ("bf16", 150, 8_000, 1_096, 64),    # ... a last stage of 8 elements
])
def test_order_is_that_of_the_distances_given(dtype, B, N, d, k):
    """Rows so near one another that rounding decides many places: the
    neighbours are the first k under (distance, index) with the very distances
    the search gives each row when it returns all of them (a bank of 64 rows,
    64 neighbours)."""
    import paper_2606_17949_amd as rb
    g = torch.Generator(device=DEV).manual_seed(9)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    centre = torch.randn(1, d, generator=g, device=DEV)
    make = lambda n: (centre + 3e-3 * torch.randn(n, d, generator=g, device=DEV)).to(t)
    q, bank = make(B), make(N)
    norms = rb.rb_bank_norms(bank)
    label = f"order of the distances {dtype} B={B} N={N} d={d} k={k}"
    print(label, flush=True)
    D = torch.empty(B, N, device=DEV)
    for r0 in range(0, N, 64):
        r1 = min(N, r0 + 64)
        i, v = rb.rb_knn_topk(q, bank[r0:r1], norms[r0:r1], r1 - r0)
        D[:, r0:r1].scatter_(1, i.long(), v)
    idx, dist = rb.rb_knn_topk(q, bank, norms, k)
    torch.cuda.synchronize()
    ref = torch.sort(D, dim=1, stable=True)
    assert torch.equal(dist, ref.values[:, :k]), label
    assert torch.equal(idx, ref.indices[:, :k].to(torch.int32)), label
