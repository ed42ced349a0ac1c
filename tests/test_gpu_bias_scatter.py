"""The gradient of the bias table where an entry's contributions do not fill the 16 lanes that add them, fill them exactly
and take several turns, and where the last workgroup is cut: against sums in 64 bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,k", [(1, 1), (3, 3), (1, 4), (5, 5), (32, 7), (2, 13), (1, 16)])
def test_scatter(heads, k):
    import torch
    import paper_2501_06480_amd as fwa
    L, W = k * k, 2 * k - 1
    db = np.random.default_rng(100 * heads + k).standard_normal((heads, L, L)).astype(np.float32)
    at = np.stack([np.arange(L) // k, np.arange(L) % k])
    dy, dx = at[:, :, None] - at[:, None, :] + k - 1
    want = np.zeros((heads, W * W))
    bound = np.zeros((heads, W * W))
    for h in range(heads):
        np.add.at(want[h], (dy * W + dx).reshape(-1), db[h].reshape(-1).astype(np.float64))
        np.add.at(bound[h], (dy * W + dx).reshape(-1), np.abs(db[h]).reshape(-1).astype(np.float64))
    got = [fwa.fwa_bias_scatter(torch.from_numpy(db).cuda(), k).cpu().numpy() for _ in range(2)]
    # at most 16 additions in a row and four levels of the tree, each rounding once by 2^-24 of a partial sum
    assert (np.abs(got[0] - want) <= 20 * 2.0 ** -24 * bound).all()
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("heads,k", [(1, 1), (3, 2), (29, 3), (5, 7), (12, 8), (7, 9), (33, 12), (40, 16), (2100, 4)])
def test_gather(oracle, heads, k):
    """One row per workgroup and up to 256 of them, the last workgroup cut, whole and ragged powers of two of columns, several turns of
    a workgroup (more rows than 8192 workgroups hold)."""
    import torch
    import paper_2501_06480_amd as fwa
    table = np.random.default_rng(200 * heads + k).standard_normal((heads, (2 * k - 1) ** 2)).astype(np.float32)
    assert np.array_equal(fwa.fwa_bias_gather(torch.from_numpy(table).cuda(), k).cpu().numpy(), oracle.bias_gather(table, k).astype(np.float32))


def test_more_entries_than_a_launch_has_room_for():
    """16 lanes per entry of 2^28 + 5 entries are more threads than one launch holds."""
    import torch
    import paper_2501_06480_amd as fwa
    heads = 2 ** 28 + 5
    db = torch.arange(heads, dtype=torch.float32, device="cuda").view(heads, 1, 1)
    assert torch.equal(fwa.fwa_bias_scatter(db, 1).view(-1), db.view(-1))
