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
