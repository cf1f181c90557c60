"""Grouping at the sizes where its shape changes: tiles of 2048 keys, four tiles per counting workgroup beyond 65 536 keys,
one to three passes of up to twelve bits (kernels for up to nine bits and for more).  Integers: exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def grouped(keys):
    perm = np.argsort(keys, kind="stable")
    unique, start = np.unique(keys[perm], return_index=True)
    return unique, np.append(start, len(keys)), perm


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, 12_345, 65_537, 300_001])
@pytest.mark.parametrize("bits", [1, 9, 10, 12, 13, 21, 22, 23, 31])
def test_groups_of_any_length_and_key_width(n, bits):
    import paper_1806_03925_amd as g
    st = g.GearState(g.make_config(16, 16, 16, 8, 8, (8, 1), max_batch=1, max_nnz=n))
    rng = np.random.default_rng(n + bits)
    span = (1 << bits) - 1
    keys = np.minimum((rng.random(n) ** 6 * span).astype(np.int64), span - 1 if bits > 1 else 1).astype(np.int32)
    keys[rng.integers(0, n, n // 2)] = keys[n // 2]           # a run over many tiles
    keys[-1] = span                                           # the widest key there is
    print(f"group n {n} bits {bits}", flush=True)
    for _ in range(2):                                        # the second time on whatever the first left behind
        unique, segoff, perm, n_unique = g.gear_group_ids(st, torch.from_numpy(keys).cuda(), 1 << bits)
        ru, rs, rp = grouped(keys)
        m = int(n_unique.item())
        assert m == len(ru)
        assert np.array_equal(unique[:m].cpu().numpy(), ru)
        assert np.array_equal(segoff[:m + 1].cpu().numpy(), rs)
        assert np.array_equal(perm.cpu().numpy(), rp)
