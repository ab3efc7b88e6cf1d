"""CPU-only: which kernels a call launches and what memory they are handed, taken from the library
itself with a recorder in the place of the HIP runtime (tests/launch_recorder.py)."""
import pytest

from paper_2603_14360_amd import binding as mb
import launch_recorder as lr

WS = 0x10000000
BF16, F32 = mb.M2RNN_BF16, mb.M2RNN_F32


def d(B, T, N, K, V, io, **kw):
    return dict(B=B, T=T, N=N, K=K, V=V, io=io, **kw)


def ws_bytes(desc, bwd):
    return mb.m2rnn_workspace_bytes(mb.make_desc(**desc), bwd)


# every shape with a split forward that can also do without a workspace
NO_WORKSPACE = [(64, 32, 4), (64, 32, 70), (32, 16, 3), (32, 16, 200), (32, 32, 300), (16, 16, 40), (64, 64, 600)]


@pytest.mark.parametrize("K,V,units", NO_WORKSPACE)
def test_a_missing_workspace_is_never_written(K, V, units):
    """workspace = NULL with a size beside it (an allocation that failed, say): where the call can
    do without a workspace it takes a split without partial sums."""
    desc = d(units, 40, 1, K, V, BF16)
    null, none, full = lr.launches([dict(call="fwd", desc=desc, ws=None, ws_bytes=1 << 30),
                                    dict(call="fwd", desc=desc, ws=None, ws_bytes=0),
                                    dict(call="fwd", desc=desc, ws=WS, ws_bytes=1 << 30)])
    assert null["rc"] == none["rc"] == full["rc"] == 0
    assert null["launches"] == none["launches"]
    assert [l["kernel"].split("<")[0] for l in null["launches"]] in (["half_fwd_kernel"], ["rowwave_fwd_kernel"])
    for l in full["launches"]:
        assert l["partial"] in (None, WS)
