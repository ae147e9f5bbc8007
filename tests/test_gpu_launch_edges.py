"""Sizes at which a launch rule changes: one case on either side of each line,
and the inputs that a rule's special path has to get right."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_32420_amd as P

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _mask_rows_admissible(got, want, fragile, alts_of):
    for (b, h, i) in np.argwhere((got != want).any(axis=-1)):
        key = (int(b), int(h), int(i))
        assert key in fragile, key
        assert any(np.array_equal(got[b, h, i] != 0, a) for a in alts_of(fragile[key])), key


# Rows of 64 E blocks and one block either side (E positions per lane), at a
# scale of 30: the logits of a row then span more than 800, so most weights
# are below the subnormals and some rows keep a single block.
@pytest.mark.parametrize("nb", [64, 65, 128, 129, 511, 513, 640, 641, 1024, 1025, 1536, 1537])
@pytest.mark.parametrize("scale", [30.0, 0.0])
def test_selection_at_row_padding_edges(nb, scale):
    print("selection edge", nb, scale, flush=True)
    g = torch.Generator(device=DEV).manual_seed(nb)
    n = nb * 64 - 5
    qh = torch.randn(1, 1, n, 64, generator=g, device=DEV) + 2.0 * torch.randn(1, 1, 1, 64, generator=g, device=DEV)
    kh = torch.randn(1, 1, n, 64, generator=g, device=DEV) * 4.0
    qh, kh = qh.to(torch.bfloat16), kh.to(torch.bfloat16)
    got = P.build_block_mask(qh, kh, 64, 0.9, scale=scale)
    want, rep = oracle.build_block_mask(oracle.to_f64(qh), oracle.to_f64(kh), 64, 0.9, scale=scale or None)
    fragile = {k: rep["scores"][k] for k in rep["fragile"]}
    _mask_rows_admissible(got.cpu().numpy(), want, fragile, lambda s: oracle.row_admissible_masks(s, 0.9))


# Ties that start in one 64-block word and end in another: the lower indices
# of the tied run are kept, also where the last one falls on a word boundary.
@pytest.mark.parametrize("nb,first,last,keep", [(200, 60, 70, 4), (200, 60, 130, 5), (640, 63, 577, 66),
                                                (1100, 0, 1099, 64), (1100, 0, 1099, 65)])
def test_selection_ties_across_words(nb, first, last, keep):
    mass = np.full((1, 1, nb, nb), 1e-5)
    mass[..., first:last + 1] = 1.0
    # a threshold reached by `keep` of the tied blocks and by no fewer
    tau = (keep - 0.5) / mass[0, 0, 0].sum()
    got = P.select_block_mask(torch.as_tensor(mass, device=DEV), float(tau))
    want = np.zeros(nb, np.uint8)
    want[first:first + keep] = 1
    assert (got.cpu().numpy() == want).all()
    bits = P.select_block_mask(torch.as_tensor(mass, device=DEV), float(tau), bits=True)
    np.testing.assert_array_equal(bits.cpu().numpy().view(np.uint64), oracle.pack_mask(got.cpu().numpy()))


# The exact masses around the pass's fixed reference: logits whose later keys
# exceed the first 32 by more than 2^100 (the workgroup starts over with the row
# maxima) or whose keys all lie far below 0, beside ordinary ones; grids of 4-
# and of 8-wave workgroups.  Scores are fp32 sums of D bf16
# products in 3 to 8 roundings of 2^-24 |x|: with |x| up to 600 log2 units a
# mass is off by 600 * 8 * 6e-8 = 3e-4 relative at most.
@pytest.mark.parametrize("kind", ["plain", "rising", "low", "mixed"])
@pytest.mark.parametrize("n,heads,d,bs", [(31, 1, 128, 64), (321, 2, 64, 64), (700, 2, 128, 128), (4161, 1, 64, 128),
                                          (1100, 90, 128, 64), (1030, 90, 64, 64),
                                          (500, 256, 128, 128)])
def test_exact_mass_reference_and_workgroup_sizes(kind, n, heads, d, bs):
    print("exact mass", kind, n, heads, d, bs, flush=True)
    g = torch.Generator(device=DEV).manual_seed(n)
    q = torch.randn(1, heads, n, d, generator=g, device=DEV)
    k = torch.randn(1, heads, n, d, generator=g, device=DEV)
    q[..., 0] = 20.0
    t = torch.arange(n, device=DEV, dtype=torch.float32)
    root = d ** 0.5 / 20.0  # k[..., 0] = root * y shifts a logit by y
    if kind == "rising":
        k[..., 0] = root * 300.0 * t / n
    elif kind == "low":
        k[..., 0] = -root * 250.0
    elif kind == "mixed":
        k[..., 0] = root * torch.where(t % 97 == 96, 200.0, -150.0)
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    mass = P.block_mass_exact(q, k, bs).cpu().numpy()
    nb = -(-n // bs)
    rows = sorted({(0, h, i) for h in (0, heads - 1) for i in (0, nb // 2, nb - 1)})
    for (b, h, i) in rows:
        ref = oracle.exact_block_mass(oracle.to_f64(q[:, h:h + 1]), oracle.to_f64(k[:, h:h + 1]), bs, rows=[(b, 0, i)])
        want = ref[b, 0, i]
        assert np.abs(mass[b, h, i] - want).max() <= 3e-4 * want.max(), (h, i)
    np.testing.assert_allclose(mass.sum(-1), 1.0, atol=1e-6)


# Attention around the one reference per query (the largest score of the first
# stage's 32 or 64 keys, below 0 raised by 32 up to 0): logits whose later keys
# exceed it by 2^60 (in range), by more than 2^100 or 2^128 (the workgroup
# walks the row again under running maxima), all 30 below 0 (reference 0) or
# 250 (a reference below 0), or mixed between the workgroup's queries (walked
# again); values near the largest bf16, whose products overflow beside a grown
# reference.
# Logits here reach 600 in log2 units and carry up to D / 16 + 1 fp32
# roundings of 2^-24 of that each: 3e-4 relative on a probability, far below
# the bf16 rounding of P and O (2^-8 each) that the tolerances are for.
@pytest.mark.parametrize("kind", ["plain", "rise60", "rise120", "rise300", "low", "low30", "mixed", "huge"])
@pytest.mark.parametrize("n,d,bs", [(1000, 128, 128), (1000, 64, 128), (690, 128, 64), (690, 64, 64), (40, 64, 128),
                                    (50, 64, 64), (70, 64, 64), (150, 64, 64)])
def test_attention_reference_range(kind, n, d, bs):
    print("attention reference", kind, n, d, bs, flush=True)
    g = torch.Generator(device=DEV).manual_seed(n + d)
    q, k, v = (torch.randn(1, 2, n, d, generator=g, device=DEV) for _ in range(3))
    t = torch.arange(n, device=DEV, dtype=torch.float32)
    q[..., 0] = 20.0
    unit = d ** 0.5 / 20.0 * 0.6931  # k[..., 0] = unit * y shifts a logit by y in log2 units
    if kind.startswith("rise"):
        k[..., 0] = unit * float(kind[4:]) * t / n
    elif kind.startswith("low"):
        k[..., 0] = -unit * float(kind[3:] or 250)
    elif kind == "mixed":
        k[..., 0] = unit * torch.where(t % 97 == 96, 200.0, -150.0)
        q[..., 0] = torch.where(t % 3 == 0, 20.0, 1.0)
    elif kind == "huge":
        k[..., 0] = unit * 90.0 * t / n
        v *= 2.0 ** 100
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    nb = -(-n // bs)
    m = (np.random.default_rng(n).random((1, 2, nb, nb)) < 0.5).astype(np.uint8)
    m[..., -1] |= m.sum(-1) == 0
    m[0, 0, :, -1] = 1  # the partial block in every list of one head
    dm = torch.as_tensor(m, device=DEV)
    o, lse = P.block_sparse_attn(q, k, v, dm, bs, return_lse=True)
    assert torch.equal(o, P.block_sparse_attn(q, k, v, dm, bs))
    ro, rl = oracle.block_sparse_attention(oracle.to_f64(q), oracle.to_f64(k), oracle.to_f64(v), m, bs)
    got = o.double().cpu().numpy()
    unit_v = 2.0 ** 100 if kind == "huge" else 1.0
    assert np.abs(got - ro).max() <= 2e-2 * unit_v * max(1.0, np.abs(ro).max() / unit_v / 2)
    assert np.linalg.norm(got - ro) <= 5e-3 * np.linalg.norm(ro)
    assert np.abs(lse.double().cpu().numpy() - rl).max() <= 1e-3


# Inputs that are not finite give what they gave under running maxima: an
# infinite value reaches exactly the queries whose lists hold it.
def test_attention_infinite_values():
    n, d, bs = 600, 128, 128
    g = torch.Generator(device=DEV).manual_seed(5)
    q, k, v = (torch.randn(1, 1, n, d, generator=g, device=DEV).to(torch.bfloat16) for _ in range(3))
    v[0, 0, 200, 7] = float("inf")  # key block 1
    m = np.ones((1, 1, 5, 5), np.uint8)
    m[0, 0, ::2, 1] = 0
    o = P.block_sparse_attn(q, k, v, torch.as_tensor(m, device=DEV), bs)
    seen = torch.isinf(o[0, 0, :, 7])
    holds = torch.arange(n, device=DEV) // bs % 2 == 1
    assert torch.equal(seen, holds)
    assert torch.isfinite(o[0, 0][:, torch.arange(d, device=DEV) != 7]).all()
    clean = v.clone()
    clean[0, 0, 200, 7] = 0
    want = P.block_sparse_attn(q, k, clean, torch.as_tensor(m, device=DEV), bs)
    assert torch.equal(o[0, 0, ~holds], want[0, 0, ~holds])


# Compaction of few rows in one launch: up to 128 words of 64 key blocks from
# bytes and 256 from bits, and one more of either; one and several words per
# row, empty and full rows.
@pytest.mark.parametrize("batch,heads,nb", [(1, 1, 1), (1, 1, 2), (2, 3, 3), (1, 128, 1), (1, 129, 1), (1, 256, 1),
                                            (1, 257, 1), (1, 2, 64), (2, 2, 64), (1, 5, 64), (1, 1, 65), (1, 2, 65),
                                            (1, 1, 128), (1, 1, 129), (2, 6, 16), (1, 8, 16)])
@pytest.mark.parametrize("density", [0.0, 0.3, 1.0])
def test_compaction_of_few_rows(batch, heads, nb, density):
    rng = np.random.default_rng(1000 * nb + heads)
    m = (rng.random((batch, heads, nb, nb)) < density).astype(np.uint8) * np.uint8(3)
    m[0, 0, nb // 2] = 0
    m[-1, -1, -1] = 1
    one = (m != 0).astype(np.uint8)

    def same(got, want):
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a.cpu().numpy()[:len(b)], b)

    dm = torch.as_tensor(m, device=DEV)
    same(P.compact_block_mask(dm), oracle.compact_mask(one))
    packed = oracle.pack_mask(one)
    if nb % 64:
        packed[..., -1] |= np.uint64(1) << np.uint64(63)  # an unused bit: ignored
    bits = torch.as_tensor(packed.view(np.int64), device=DEV)
    same(P.compact_block_mask_bits(bits), oracle.compact_mask(one))
    rows = (rng.random((batch, nb)) < 0.2).astype(np.uint8)
    cols = (rng.random((batch, nb)) < 0.1).astype(np.uint8)
    same(P.compact_block_mask_bits(bits, rows, cols), oracle.compact_mask(oracle.merge_target_rows(one, rows, cols)))
    for act in (rows, np.zeros_like(rows), np.ones_like(rows)):
        ctx = np.maximum(act, cols)
        got = P.compact_block_mask_bits_region(bits, act, ctx)
        want = oracle.compact_restricted(one, act, ctx)
        same(got[:3], want[:3])
        assert int(got[3].item()) == want[3]


# Lists from packed rows counted beside the sort's histograms (up to four words
# a row, more rows than one launch takes) and by a launch of their own, with
# chunks of rows that span many batch entries and entries that span chunks.
@pytest.mark.parametrize("batch,heads,nb", [(1, 257, 1), (1100, 1, 1), (300, 1, 5), (40, 1, 30), (3, 7, 64), (2, 9, 65),
                                            (1, 3, 193), (2, 5, 256), (1, 2, 257), (2, 5, 300)])
def test_compaction_from_bits_count(batch, heads, nb):
    rng = np.random.default_rng(nb + batch)
    m = (rng.random((batch, heads, nb, nb)) < 0.3).astype(np.uint8)
    m[0, 0, nb // 2] = 0
    packed = oracle.pack_mask(m)
    if nb % 64:
        packed[..., -1] |= np.uint64(1) << np.uint64(63)  # an unused bit: ignored
    bits = torch.as_tensor(packed.view(np.int64), device=DEV)
    rows = (rng.random((batch, nb)) < 0.3).astype(np.uint8)
    cols = (rng.random((batch, nb)) < 0.2).astype(np.uint8) * np.uint8(7)
    group = P.order_group_heads(batch, heads, nb)

    def same(got, want):
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a.cpu().numpy()[:len(b)], b)

    for r, c in ((None, None), (rows, None), (None, cols), (rows, cols)):
        same(P.compact_block_mask_bits(bits, r, c), oracle.compact_mask(oracle.merge_target_rows(
            m, np.zeros_like(rows) if r is None else r, c), group_heads=group))
    ctx = np.maximum(rows, cols)
    got, want = P.compact_block_mask_bits_region(bits, rows, ctx), oracle.compact_restricted(m, rows, ctx, group_heads=group)
    same(got[:3], want[:3])
    assert int(got[3].item()) == want[3]


# The same from a row order of several head groups: chunks that start at a
# group's first row, partial chunks inside the grid, and batch entries that
# begin in the middle of a group or of a chunk.
@pytest.mark.parametrize("batch,heads,nb,attn", [(1, 40, 256, (32760, 128, 128)), (2, 24, 256, (32760, 128, 128)),
                                                 (3, 40, 193, (193 * 128 - 7, 128, 128)),
                                                 (1, 260, 129, (129 * 64, 64, 64))])
def test_compaction_from_bits_count_of_head_groups(batch, heads, nb, attn):
    rng = np.random.default_rng(nb + heads)
    m = (rng.random((batch, heads, nb, nb)) < 0.3).astype(np.uint8)
    m[0, 0, nb // 2] = 0
    bits = torch.as_tensor(oracle.pack_mask(m).view(np.int64), device=DEV)
    rows = (rng.random((batch, nb)) < 0.3).astype(np.uint8)
    cols = (rng.random((batch, nb)) < 0.2).astype(np.uint8)
    group = P.order_group_heads(batch, heads, nb, attn=attn)
    assert group < batch * heads

    def same(got, want):
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a.cpu().numpy()[:len(b)], b)

    for r, c in ((None, None), (rows, cols)):
        same(P.compact_block_mask_bits(bits, r, c, attn=attn), oracle.compact_mask(oracle.merge_target_rows(
            m, np.zeros_like(rows) if r is None else r, c), group_heads=group))
    ctx = np.maximum(rows, cols)
    got = P.compact_block_mask_bits_region(bits, rows, ctx, attn=attn)
    want = oracle.compact_restricted(m, rows, ctx, group_heads=group)
    same(got[:3], want[:3])
    assert int(got[3].item()) == want[3]


# A value that is not finite reaches exactly the queries whose lists hold its
# key block, also where a stage reaches past the last token: in the block
# before the ragged one, whose rows such a stage's tile takes in; in the ragged
# block itself, which a second half-stage past the end takes in again; and with
# fewer tokens than a stage, where the rows past the end repeat the last one.
@pytest.mark.parametrize("n,d,bs,token", [(600, 64, 64, 550), (600, 128, 64, 570), (540, 128, 128, 500),
                                          (540, 64, 128, 480), (540, 128, 128, 520), (540, 64, 128, 539),
                                          (610, 128, 64, 585), (40, 64, 128, 39), (20, 128, 64, 19), (50, 64, 64, 49)])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_attention_infinite_values_near_the_end(n, d, bs, token, bad):
    print("attention non-finite value", n, d, bs, token, bad, flush=True)
    g = torch.Generator(device=DEV).manual_seed(n + d)
    q, k, v = (torch.randn(1, 1, n, d, generator=g, device=DEV).to(torch.bfloat16) for _ in range(3))
    clean = v.clone()
    v[0, 0, token, 7] = bad
    nb = -(-n // bs)
    m = np.ones((1, 1, nb, nb), np.uint8)
    if nb > 1:
        m[0, 0, ::2, token // bs] = 0
    holds = torch.arange(n, device=DEV) // bs % 2 == 1 if nb > 1 else torch.ones(n, dtype=torch.bool, device=DEV)
    dm = torch.as_tensor(m, device=DEV)
    o, _ = P.block_sparse_attn(q, k, v, dm, bs, return_lse=True)
    assert torch.equal(o.isfinite(), P.block_sparse_attn(q, k, v, dm, bs).isfinite())
    o = o[0, 0]
    hit = torch.isinf(o[:, 7]) if bad == float("inf") else torch.isnan(o[:, 7])
    assert torch.equal(hit, holds)
    assert torch.isfinite(o[:, torch.arange(d, device=DEV) != 7]).all()
    want = P.block_sparse_attn(q, k, clean, dm, bs)[0, 0]
    assert torch.equal(o[~holds], want[~holds])


def _shifted(heads, n, d, base, rise, seed=0):
    """q, k, v with base + rise t / n (log2 units) added to every logit of key t."""
    g = torch.Generator(device=DEV).manual_seed(n + d + seed)
    q, k, v = (torch.randn(1, heads, n, d, generator=g, device=DEV) for _ in range(3))
    q[..., 0] = 20.0
    t = torch.arange(n, device=DEV, dtype=torch.float32)
    k[..., 0] = d ** 0.5 / 20.0 * 0.6931 * (base + rise * t / n)
    return (x.to(torch.bfloat16) for x in (q, k, v))


# Logits below 0: every one lower by the same amount (either side of the line
# below which a query's reference follows its scores), and scores that climb
# from there by less than a reference below 0 allows, or by more (the workgroup
# starts over).  Logits reach 140 log2 units over up to D / 16 + 2 roundings of
# 2^-24 of that each, and x - r rounds by 2^-19 at most: 9e-5 in log2 units,
# 6e-5 in the LSE and on a mass relative to its row's largest.
_CLIMBS = [(-20.0, 0.0), (-31.0, 0.0), (-35.0, 0.0), (-60.0, 0.0), (-110.0, 0.0), (-60.0, 40.0), (-60.0, 80.0),
           (-100.0, 80.0), (-100.0, 90.0), (-100.0, 120.0), (-20.0, 130.0)]


@pytest.mark.parametrize("base,rise", _CLIMBS)
@pytest.mark.parametrize("n,d,bs", [(1000, 128, 128), (1000, 64, 128), (690, 128, 64), (690, 64, 64), (50, 64, 64)])
def test_attention_reference_below_zero(base, rise, n, d, bs):
    print("attention reference", base, rise, n, d, bs, flush=True)
    q, k, v = _shifted(2, n, d, base, rise)
    nb = -(-n // bs)
    m = np.ones((1, 2, nb, nb), np.uint8)
    dm = torch.as_tensor(m, device=DEV)
    o, lse = P.block_sparse_attn(q, k, v, dm, bs, return_lse=True)
    assert torch.equal(o, P.block_sparse_attn(q, k, v, dm, bs))
    ro, rl = oracle.block_sparse_attention(oracle.to_f64(q), oracle.to_f64(k), oracle.to_f64(v), m, bs)
    got = o.double().cpu().numpy()
    assert np.abs(got - ro).max() <= 2e-2
    assert np.linalg.norm(got - ro) <= 5e-3 * np.linalg.norm(ro)
    err = float(np.abs(lse.double().cpu().numpy() - rl).max())
    print("lse error", err)
    assert err <= 6e-5


@pytest.mark.parametrize("base,rise", _CLIMBS)
@pytest.mark.parametrize("n,heads,d,bs", [(700, 2, 128, 128), (321, 2, 64, 64), (1030, 90, 64, 64)])
def test_exact_mass_reference_below_zero(base, rise, n, heads, d, bs):
    print("exact mass reference", base, rise, n, heads, d, bs, flush=True)
    q, k, _ = _shifted(heads, n, d, base, rise)
    mass = P.block_mass_exact(q, k, bs).cpu().numpy()
    nb = -(-n // bs)
    for (h, i) in sorted({(h, i) for h in (0, heads - 1) for i in (0, nb // 2, nb - 1)}):
        want = oracle.exact_block_mass(oracle.to_f64(q[:, h:h + 1]), oracle.to_f64(k[:, h:h + 1]), bs,
                                       rows=[(0, 0, i)])[0, 0, i]
        assert np.abs(mass[0, h, i] - want).max() <= 6e-5 * want.max(), (h, i)
    np.testing.assert_allclose(mass.sum(-1), 1.0, atol=1e-6)


def _times(calls, repeats=15):
    """Median time of each call (us), the calls taken in turn."""
    took = [[] for _ in calls]
    for i in range(repeats + 3):
        for c, t in zip(calls, took):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            c()
            b.record()
            b.synchronize()
            if i >= 3:
                t.append(1e3 * a.elapsed_time(b))
    return [float(np.median(t)) for t in took]


# One amount taken from every logit leaves the softmax as it is, and costs
# nothing: a query's reference follows its scores down.  Nor do scores that
# climb from far below 0 to about 0.  A second walk of the row would be twice
# the time.
@pytest.mark.parametrize("n,d,bs", [(6000, 128, 128), (6000, 64, 128), (6000, 128, 64), (6000, 64, 64)])
@pytest.mark.parametrize("base,rise", [(-20.0, 0.0), (-60.0, 0.0), (-300.0, 0.0), (-60.0, 60.0), (-90.0, 80.0)])
def test_attention_time_of_shifted_logits(n, d, bs, base, rise):
    heads, nb = 24, -(-n // bs)
    lists = P.compact_block_mask(torch.ones(1, heads, nb, nb, dtype=torch.uint8, device=DEV))
    calls = []
    for shift, up in ((0.0, 0.0), (base, rise)):
        q, k, v = _shifted(heads, n, d, shift, up)
        calls.append(lambda q=q, k=k, v=v: P.block_sparse_attn_lists(q, k, v, lists, bs))
    plain, shifted = _times(calls)
    print("attention", n, d, bs, base, rise, "plain %.1f us, shifted %.1f us" % (plain, shifted), flush=True)
    assert shifted <= 1.35 * plain


@pytest.mark.parametrize("n,d,bs", [(6000, 128, 128), (6000, 64, 64)])
@pytest.mark.parametrize("base,rise", [(-20.0, 0.0), (-60.0, 0.0), (-300.0, 0.0), (-60.0, 60.0), (-90.0, 80.0)])
def test_exact_mass_time_of_shifted_logits(n, d, bs, base, rise):
    calls = []
    for shift, up in ((0.0, 0.0), (base, rise)):
        q, k, _ = _shifted(24, n, d, shift, up)
        calls.append(lambda q=q, k=k: P.block_mass_exact(q, k, bs))
    plain, shifted = _times(calls)
    print("exact mass", n, d, bs, base, rise, "plain %.1f us, shifted %.1f us" % (plain, shifted), flush=True)
    assert shifted <= 1.35 * plain


# A reference and a row sum that are both large beside the LSE: the keys of the
# first stage lie 60 to 84 log2 units below 0, four later ones at exactly 0, so
# the LSE is log 4.  Roundings of 2^-24: one in the exponential (two as an ulp),
# three in the sum, two in the mantissa's log2, and one of an LSE of 1.4: 8 of
# 6e-8 at most.
@pytest.mark.parametrize("d,bs", [(128, 128), (64, 128), (128, 64), (64, 64)])
def test_attention_lse_beside_a_large_reference(d, bs):
    n = 68
    q, k = torch.zeros(1, 1, n, d, device=DEV), torch.zeros(1, 1, n, d, device=DEV)
    q[0, 0, :, 0] = 20.0 + 0.125 * torch.arange(n, device=DEV) % 8.0
    k[0, 0, :64, 0] = -3.0 * 0.6931 * d ** 0.5
    nb = -(-n // bs)
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    _, lse = P.block_sparse_attn(q, k, torch.ones_like(q), torch.ones(1, 1, nb, nb, dtype=torch.uint8, device=DEV), bs,
                                 return_lse=True)
    err = float((lse.double() - np.log(4.0)).abs().max())
    print("lse error", d, bs, err)
    assert err <= 5e-7


# d = 64 with 64-token blocks takes stages of a whole block or of half of one
# by the number of rows (768, 7680) and of key blocks (120): each side of each
# line, with a ragged last block and an infinite value in the block before it
# that half of the lists leave out; logits as they are, climbing by 130 log2
# units (walked twice) and all 60 lower.  P and O are rounded to bf16 (2^-9 each
# of values up to 4), the LSE carries fp32 roundings only (as above).
@pytest.mark.parametrize("base,rise", [(0.0, 0.0), (0.0, 130.0), (-60.0, 0.0)])
@pytest.mark.parametrize("heads,n", [(768, 40), (769, 40), (256, 190), (257, 190), (64, 120 * 64 - 9),
                                     (63, 120 * 64 - 9), (65, 119 * 64 - 9)])
def test_attention_stage_rule(heads, n, base, rise):
    print("attention stages", heads, n, base, rise, flush=True)
    d = bs = 64
    nb = -(-n // bs)
    g = torch.Generator(device=DEV).manual_seed(n + heads)
    q, k, v = _shifted(heads, n, d, base, rise)
    m = (torch.rand(1, heads, nb, nb, generator=g, device=DEV) < 0.1).to(torch.uint8)
    m[..., -1] = 1
    if nb > 1:
        v[..., (nb - 1) * bs - 3, 7] = float("inf")
        m[..., ::2, nb - 2] = 0
        m[..., 1::2, nb - 2] = 1
    o, lse = P.block_sparse_attn(q, k, v, m, bs, return_lse=True)
    holds = (torch.arange(n, device=DEV) // bs % 2 == 1) & (nb > 1)
    assert torch.equal(torch.isinf(o[..., 7]), holds.expand(1, heads, n))
    o[..., 7] = v[..., 7] = 0
    assert torch.isfinite(o).all()
    v = v.double()
    for h in (0, heads // 2, heads - 1):
        for i in (0, nb // 2, nb - 1):
            rows = slice(i * bs, min((i + 1) * bs, n))
            keep = m[0, h, i].repeat_interleave(bs)[:n].bool().cpu()
            x = (q[0, h, rows].double().cpu() @ k[0, h].double().cpu().T.contiguous()) / d ** 0.5
            x = x.masked_fill(~keep, float("-inf"))
            want = torch.softmax(x, -1) @ v[0, h].cpu()
            assert (o[0, h, rows].double().cpu() - want).abs().max() <= 2e-2
            assert (lse[0, h, rows].double().cpu() - torch.logsumexp(x, -1)).abs().max() <= 6e-5


# One third more rows than three workgroups per CU take a third more time, not
# a second round: 12 and 16 heads of 63 rows, a band of 30 % of the pairs.
def test_attention_time_past_three_workgroups_per_cu():
    n, d, bs, nb = 4000, 64, 64, 63
    i = torch.arange(nb, device=DEV)
    band = ((i[:, None] - i[None]).abs() <= 0.15 * nb).to(torch.uint8)
    calls = []
    for heads in (12, 16):
        q, k, v = _shifted(heads, n, d, 0.0, 0.0)
        lists = P.compact_block_mask(band.expand(1, heads, nb, nb).contiguous())
        calls.append(lambda q=q, k=k, v=v, lists=lists: [P.block_sparse_attn_lists(q, k, v, lists, bs) for _ in range(20)])
    a, b = _times(calls)
    print("attention 12 heads %.1f us, 16 heads %.1f us" % (a / 20, b / 20), flush=True)
    assert b <= 1.5 * a
