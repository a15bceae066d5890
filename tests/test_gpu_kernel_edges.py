"""Kernels at the sizes where a tile, a split or a bank can go wrong: edges,
remainders, and the smallest and largest of a rule's range."""
import numpy as np
import pytest
import torch

from paper_2603_04035_amd import datagen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [12, 129, 5000])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_update_count_over_counter_banks(n, precision):
    """The update count (summed over the counter banks by the host) equals
    the entries of the merged lists that the initial lists did not hold, with
    fewer joined points than banks, about as many, and many more."""
    import paper_2603_04035_amd as knn
    X = torch.from_numpy(datagen.gmm_isotropic(n=n, d=20, seed=n)).cuda()
    states = []
    for iters in (0, 1):
        _, _, st, (idx, _, _) = knn.nndescent_build(X, 5, build_k=8, sample_rate=1.0, max_iters=iters, delta=0.0,
                                                    seed=3, precision=precision, return_state=True)
        states.append(idx.cpu().numpy())
    new = ~(states[1][:, :, None] == states[0][:, None, :]).any(2) & (states[1] >= 0)
    assert st["iters"] == 1 and st["updates"][0] == int(new.sum())
    assert st["emitted"][0] >= st["updates"][0] and st["pairs_joined"] > 0
