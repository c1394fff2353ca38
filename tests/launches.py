"""How many kernels a call launches: the call recorded into a HIP graph, which is not run."""
import ctypes

import torch

import paper_2108_02191_amd as robe


def kernels(call):
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    n = ctypes.c_size_t(0)
    assert robe.lib().hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value
