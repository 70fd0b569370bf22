"""GPU parity of middle-channel pruning (section 3.5; dbf_prune_middle): the pruned layer, read back
through dbf_unpack_bits, must equal the oracle's prune_middle BIT FOR BIT (signs, m; a and b
unchanged), its padding must be clean (the forward of the pruned layer equals the oracle's forward of
the pruned layer), and pruning must not touch the old layer.  Shapes span several tiles with ragged
tails in all three dimensions; keeps are random subsets, a prefix, a suffix, every other channel,
a single channel and the identity."""
import numpy as np
import pytest
import torch

import gpu_util as G
from oracle import dbf_oracle as O
from paper_2505_11076_amd import binding as B
from paper_2505_11076_amd import inputs as I

pytestmark = pytest.mark.gpu


def _keeps(k, rng):
    yield "random 2/3", np.sort(rng.choice(k, size=max(1, (2 * k) // 3), replace=False))
    yield "random 1/12", np.sort(rng.choice(k, size=max(1, k // 12), replace=False))
    yield "random 1/4", np.sort(rng.choice(k, size=max(1, k // 4), replace=False))
    yield "prefix", np.arange(max(1, k // 2))
    yield "suffix", np.arange(k // 3, k)
    yield "every other", np.arange(0, k, 2)
    yield "single", np.array([k - 1])
    yield "identity", np.arange(k)


# (the last two: more tiles than a workgroup takes, kept columns from one to many tiles of the old matrix, ragged groups of tiles)
@pytest.mark.parametrize("shape", [(512, 512, 256), (100, 77, 333), (1000, 130, 129), (300, 700, 1000), (650, 1300, 1500), (321, 513, 2050)])
def test_pruned_layer_equals_the_oracle_bit_for_bit(shape):
    n_in, n_out, k = shape
    L = I.make_layer(n_in, n_out, k, seed=I.seed_for(7, k))
    X = I.make_activations(3, n_in, I.seed_for(7, k + 1))
    layer = G.pack(L)
    try:
        before = B.dbf_unpack_bits(layer)
        for name, keep in _keeps(k, np.random.default_rng(I.seed_for(7, k + 2))):
            G.say("prune %s: %s (%d of %d)" % (shape, name, keep.size, k))
            A2, B2, m2, k2 = O.prune_middle(L.A_bits, L.B_bits, L.m, n_out, k, n_in, keep)
            pruned = B.dbf_prune_middle(layer, keep)
            try:
                assert B.dbf_dims(pruned)[:3] == (n_in, n_out, k2)
                gA, gB, ga, gm, gb = B.dbf_unpack_bits(pruned)
                assert np.array_equal(gA, A2), name
                assert np.array_equal(gB, B2), name
                assert np.array_equal(gm, m2), name
                assert np.array_equal(ga, np.asarray(L.a, dtype=np.uint16)) and np.array_equal(gb, np.asarray(L.b, dtype=np.uint16))
                # forward of the pruned layer (exercises its padding and its launch plan)
                Lp = I.LayerInputs(n_in, n_out, k2, A2, B2, L.a, m2, L.b)
                x = G.f16_to_dev(X)
                y = torch.full((3, n_out), float("nan"), dtype=torch.float16, device="cuda")
                B.dbf_gemv(pruned, x.data_ptr(), y.data_ptr(), 3, G.stream_handle())
                torch.cuda.synchronize()
                got = O.f16_bits_to_f64(y.cpu().view(torch.int16).numpy().view(np.uint16)).reshape(3, n_out)
                G.check(got, O.forward_from_packed(X, Lp, "dense"), "pruned forward %s %s" % (shape, name))
            finally:
                pruned.close()
        after = B.dbf_unpack_bits(layer)
        for u, v in zip(before, after):
            assert np.array_equal(u, v)
    finally:
        layer.close()


def test_prune_rejects_bad_index_lists():
    L = I.make_layer(64, 64, 100, seed=5)
    layer = G.pack(L)
    try:
        for bad in ([], [3, 3], [5, 2], [-1, 2], [0, 100], list(range(101))):
            with pytest.raises(B.DbfError):
                B.dbf_prune_middle(layer, np.array(bad, dtype=np.int32))
    finally:
        layer.close()
