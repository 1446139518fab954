"""tpc_get_tuning reports the shapes that run: the peak pass of a context, as it is
made and after other shapes were set, on small and large frames."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2208_07412_amd import tpc

pytestmark = pytest.mark.gpu

NPADS, _, _ = oracle.geometry()


class KernelNode(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p),
                ("func", ctypes.c_void_p), ("grid", ctypes.c_uint32 * 3),
                ("params", ctypes.c_void_p), ("shared", ctypes.c_uint32)]


def launches(reco, call):
    """(workgroups, threads) of the kernels that `call` enqueues, captured and not run."""
    hip, P, z = reco.lib, ctypes.c_void_p, ctypes.c_size_t
    graph, n, s = P(), z(), P(reco.stream.cuda_stream)
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(s, 2) == 0  # relaxed
    call()
    assert hip.hipStreamEndCapture(s, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (P * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    out = []
    for node in nodes:
        k = KernelNode()
        assert hip.hipGraphKernelNodeGetParams(P(node), ctypes.byref(k)) == 0
        out.append((k.grid[0], k.block[0]))
    assert hip.hipGraphDestroy(graph) == 0
    return out


def peak_workgroups(reco, T):
    """Workgroups of the peak pass (the one launch of two waves each)."""
    rng = np.random.default_rng(3)
    rows = [np.unique(rng.integers(0, T * int(NPADS[r]), 50)) for r in range(152)]
    t = np.concatenate([k // int(NPADS[r]) for r, k in enumerate(rows)]).astype(np.uint16)
    p = np.concatenate([k % int(NPADS[r]) for r, k in enumerate(rows)]).astype(np.uint16)
    rs = np.concatenate([[0], np.cumsum([len(k) for k in rows])]).astype(np.uint32)
    zs = tpc.to_device_zs(p, t, np.full(len(t), 50, np.uint16), rs, 1, T)
    cl = reco.alloc_clusters(1, T, len(t))
    got = [g for g, b in launches(reco, lambda: reco.cluster(zs, cl)) if b == 128]
    assert len(got) == 1
    return got[0]


@pytest.mark.parametrize("bins", [500, 53 * 512 + 1])
def test_peak_pass(bins):
    reco = tpc.Reco(1, bins, 1 << 14, 64, stream=torch.cuda.Stream())

    def reported():
        t = reco.tuning()
        return 152 * -(-(-(-bins // t["cl_window"])) // t["cl_chunk"])

    assert peak_workgroups(reco, bins) == reported()
    reco.set_tuning(refit_waves=5)
    assert peak_workgroups(reco, bins) == reported()
    reco.set_tuning(cl_chunk=16)
    assert peak_workgroups(reco, bins) == reported()
    reco.close()
