"""The launches of a call -- kernels, grids, order -- found without a GPU (see launches.py)."""
import pytest

from launches import launches_of

QKV_8B = dict(op="forward", dtype=1, hidden=4096, n_q_heads=32, n_kv_heads=8, head_dim=128, rank=16, n_segments=4, n_slots=1024)


def kernels(call):
    assert call["status"] == 0, call
    return [l["kernel"] for l in call["launches"]]


@pytest.mark.parametrize("T", [1, 40, 64, 65, 100, 256])
def test_a_tuning_override_during_a_call_leaves_the_call_whole(T):
    """The override may be set by another host thread at any time: a call that has decided to group and shrink
    inside its projection kernel launches that kernel."""
    plain, torn, after = launches_of([dict(QKV_8B, T=T, n_adapters=4), dict(QKV_8B, T=T, n_adapters=4, tuning_during=[4, 1]),
                                      dict(QKV_8B, T=T, n_adapters=4)])
    assert len(plain["launches"]) == 2, kernels(plain)
    assert torn == plain and after == plain, (kernels(plain), kernels(torn))
