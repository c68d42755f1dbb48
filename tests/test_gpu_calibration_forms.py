"""The calibration of beta and the selection statistics at the sizes where they change form (one workgroup, several), at
odd expert counts, and on logits whose rows are not 16-byte aligned.  Counts are exact; beta within 2e-6 (fp32 result of
an fp64 exponential)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2402_14800_amd as pkg
from paper_2402_14800_amd import binding

pytestmark = pytest.mark.gpu


def logits_on_gpu(T, E, seed, offset=0, rounding=None):
    lg = np.random.Generator(np.random.PCG64(seed)).standard_normal((T, E)).astype(np.float32)
    if rounding:
        lg = (np.round(lg * rounding) / rounding).astype(np.float32)      # many ties
    buf = torch.empty(T * E + offset, dtype=torch.float32, device="cuda:0")
    view = buf[offset:].view(T, E)
    view.copy_(torch.from_numpy(lg))
    return lg, view


@pytest.mark.parametrize("T,E,offset,rounding", [
    (1, 2, 0, None), (2048, 8, 0, None), (2049, 8, 0, None), (512, 32, 0, None), (513, 32, 1, None),
    (8192, 2, 0, None), (8193, 2, 0, None), (3277, 5, 0, None), (3276, 5, 0, None), (4097, 16, 2, None),
    (2000, 8, 0, 4.0), (30001, 8, 0, 4.0), (140001, 4, 0, 2.0),
    (8192, 8, 0, 4.0), (8193, 8, 0, None), (4096, 16, 0, None), (2048, 32, 1, 4.0), (2049, 32, 0, None),
    (1536, 32, 0, None), (1537, 32, 0, None), (3072, 8, 1, None), (3073, 8, 1, 4.0), (3076, 13, 0, 4.0), (3077, 13, 0, None),
])
def test_beta_at_every_form(T, E, offset, rounding):
    lg, dev = logits_on_gpu(T, E, 31 + T, offset, rounding)
    got = float(pkg.skip_calibrate_beta(dev).item())
    ref = oracle.median_skip_ratio(lg)
    assert abs(got - ref) <= 2e-6 * ref


@pytest.mark.parametrize("T,E,offset,kernels", [
    (8192, 8, 0, 1), (4096, 16, 0, 1), (4097, 16, 0, 5), (1536, 32, 0, 1), (1537, 32, 0, 5),      # rows of whole 16 bytes
    (4000, 10, 1, 1), (4001, 10, 0, 5), (1927, 17, 0, 1), (1928, 17, 0, 5),                       # read word by word
    (3072, 8, 1, 1), (3073, 8, 1, 5), (768, 32, 2, 1), (769, 32, 2, 5),                           # and strides of 32 bytes
])
def test_beta_takes_one_launch_only_where_that_is_the_faster_form(T, E, offset, kernels):
    """Kernels of a call, counted in a captured graph: one workgroup reads rows word by word, and more than 16 experts, more
    slowly than the multi-workgroup form beyond fewer logits."""
    _, dev = logits_on_gpu(T, E, 97, offset)
    pkg.skip_calibrate_beta(dev)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        beta = pkg.skip_calibrate_beta(dev)
    nodes = ctypes.c_size_t(0)
    get_nodes = binding._lib.hipGraphGetNodes          # (resolved in the HIP runtime that the library is linked to)
    get_nodes.restype = ctypes.c_int
    assert get_nodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
    assert nodes.value == kernels
    del beta


@pytest.mark.parametrize("T,E,k,offset,rounding", [
    (1, 1, 1, 0, None), (1023, 8, 2, 0, 4.0), (1024, 8, 2, 0, None), (1025, 8, 2, 0, None), (1024, 32, 2, 0, None),
    (1025, 31, 31, 0, 2.0), (777, 9, 4, 0, None), (5000, 16, 4, 3, None), (300, 17, 17, 0, None),
])
def test_selection_statistics_at_every_form(T, E, k, offset, rounding):
    lg, dev = logits_on_gpu(T, E, 57 + T, offset, rounding)
    r = max(1, E // 2)
    count, co, mask = pkg.expert_selection_stats(dev, k, r)
    ref_count, ref_co = oracle.expert_selection_stats(lg, k)
    assert np.array_equal(count.cpu().numpy(), ref_count) and np.array_equal(co.cpu().numpy(), ref_co)
    order = sorted(range(E), key=lambda e: (-int(ref_count[e]), e))
    assert (int(mask.item()) & 0xFFFFFFFF) == sum(1 << e for e in order[:r])


@pytest.mark.parametrize("T,E,k,rounding", [(2047, 8, 2, None), (2048, 5, 3, 2.0), (2049, 8, 2, None), (512, 32, 2, None), (513, 17, 4, 4.0)])
def test_selection_statistics_around_the_one_workgroup_limit(T, E, k, rounding):
    lg, dev = logits_on_gpu(T, E, 91 + T, 0, rounding)
    count, co, mask = pkg.expert_selection_stats(dev, k, max(1, E // 2))
    ref_count, ref_co = oracle.expert_selection_stats(lg, k)
    torch.cuda.synchronize()
    assert np.array_equal(count.cpu().numpy(), ref_count) and np.array_equal(co.cpu().numpy(), ref_co)
    best = np.argsort(-ref_count, kind="stable")[:max(1, E // 2)]
    assert int(mask.item()) & 0xFFFFFFFF == sum(1 << int(e) for e in best)
