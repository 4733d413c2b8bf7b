"""The workspace of the pair sums and the MMD grows with every size, so that one
queried for the largest sets serves all smaller ones, whichever way a call of
theirs goes (host arithmetic; and on the GPU, calls with the larger sets'
workspace against the float64 oracle)."""
import itertools

import numpy as np
import pytest
import torch

from oracle import mmd as OM

SIZES = (1, 64, 65, 128, 129, 256, 257, 512, 1000, 1024, 2000, 2048, 2049, 2112, 1 << 17)
DIMS = (0, 1, 8, 64, 255, 256, 257, 512, 4096, 8192, 100000)


def _lib():
    from paper_2104_12922_amd import nebula
    return nebula.lib()


@pytest.mark.parametrize("name", ["synth_l1_pair_sum_workspace", "synth_mmd_l1_workspace"])
def test_queries_grow_with_every_size(name):
    f = getattr(_lib(), name)
    got = {k: f(*k) for k in itertools.product(SIZES, SIZES, DIMS)}
    for (n, m, d), v in got.items():
        for axis, values in ((0, SIZES), (1, SIZES), (2, DIMS)):
            k = [n, m, d]
            i = values.index(k[axis])
            if i + 1 < len(values):
                k[axis] = values[i + 1]
                assert got[tuple(k)] >= v, (n, m, d, k)


def test_mmd_covers_its_three_sums():
    L = _lib()
    for n, m, d in itertools.product(SIZES, SIZES, DIMS):
        assert L.synth_mmd_l1_workspace(n, m, d) >= max(
            L.synth_l1_pair_sum_workspace(*k) for k in ((n, m, d), (n, n, d), (m, m, d)))


@pytest.mark.gpu
@pytest.mark.parametrize("large,small", [((1000, 1000, 8), (1000, 64, 8)), ((1000, 1000, 8), (130, 70, 5)),
                                         ((2048, 2048, 64), (2000, 64, 64)),
                                         ((2048, 2048, 64), (300, 2, 64)),
                                         ((2112, 2112, 512), (2112, 1984, 512)),
                                         ((2500, 2500, 300), (257, 64, 300))])
def test_one_workspace_serves_smaller_sets(large, small):
    L = _lib()
    n, m, d = small
    g = torch.Generator().manual_seed(n + m + d)
    X, Y = (torch.randint(-9, 10, (k, d), generator=g).float() for k in (n, m))
    x, y, out = X.cuda(), Y.cuda(), torch.zeros(4, dtype=torch.float64, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    for query, call in ((L.synth_l1_pair_sum_workspace, L.synth_l1_pair_sum),
                        (L.synth_mmd_l1_workspace, L.synth_mmd_l1)):
        size = query(*large)
        ws = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        args = (x.data_ptr(), d, n, y.data_ptr(), d, m, d) if call is L.synth_l1_pair_sum else \
            (x.data_ptr(), n, y.data_ptr(), m, d)
        out.zero_()
        assert call(*args, ws.data_ptr(), size, out.data_ptr(), s) == 0
        torch.cuda.synchronize()
        got = float(out[0 if call is L.synth_l1_pair_sum else 1])
        assert got == OM.l1_distance_sum(X.double().numpy(), Y.double().numpy())   # whole numbers
        assert bool((ws[size:] == 0x5A).all())
