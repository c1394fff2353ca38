"""The Python functions refuse arguments that do not fit before anything reaches a GPU: lengths by
ValueError, devices, types and layouts by TypeError, each naming the argument.  No compute call is made."""
import pytest
import torch

import paper_2108_02191_amd as robe

M, B, F, D = 1000, 4, 3, 16


def arguments():
    h = robe.robe_init_hash(1, M, D, 4, 0)
    return {"h": h, "array": torch.zeros(M), "grad": torch.zeros(M), "state": torch.zeros(M), "ids": torch.zeros(B, F, dtype=torch.int64),
            "offsets": torch.zeros(B * F + 1, dtype=torch.int64), "grad_out": torch.zeros(B, F, D), "dims": [16, 8, 4],
            "out": torch.zeros(B, F, D), "workspace": None, "options": None}


CALLS = {
    "forward": lambda a: robe.robe_forward(a["h"], a["array"], a["ids"], a["offsets"], B, F, out=a["out"], options=a["options"]),
    "bf16": lambda a: robe.robe_forward_bf16(a["h"], a["array"], a["ids"], a["offsets"], B, F, out=a["out"]),
    "backward": lambda a: robe.robe_backward(a["h"], a["grad_out"], a["ids"], a["offsets"], B, F, a["grad"], options=a["options"]),
    "noalloc": lambda a: robe.robe_backward_noalloc(a["h"], a["grad_out"], a["ids"], a["offsets"], B, F, a["grad"]),
    "adagrad": lambda a: robe.robe_adagrad_update(a["h"], a["array"], a["state"], a["grad"], 0.1, 1e-8),
    "sgd": lambda a: robe.robe_sgd_update(a["h"], a["array"], a["grad"], 0.1),
    "fused": lambda a: robe.robe_backward_adagrad(a["h"], a["grad_out"], a["ids"], a["offsets"], B, F, a["array"], a["state"], 0.1, 1e-8,
                                                  workspace=a["workspace"] if a["workspace"] is not None else torch.zeros(8)),
    "fused_sgd": lambda a: robe.robe_backward_sgd(a["h"], a["grad_out"], a["ids"], a["offsets"], B, F, a["array"], 0.1, workspace=torch.zeros(8)),
    "mixed": lambda a: robe.robe_forward_mixed(a["h"], a["dims"], a["array"], a["ids"], a["offsets"], B),
    "mixed_backward": lambda a: robe.robe_backward_mixed(a["h"], a["dims"], torch.zeros(B, 28), a["ids"], a["offsets"], B, a["grad"]),
    "mixed_fused": lambda a: robe.robe_backward_adagrad_mixed(a["h"], a["dims"], torch.zeros(B, 28), a["ids"], a["offsets"], B, a["array"],
                                                              a["state"], 0.1, 1e-8, workspace=torch.zeros(8)),
}


@pytest.mark.parametrize("call", sorted(CALLS))
def test_tensors_off_the_gpu_are_refused_by_name(call):
    with pytest.raises(TypeError, match="need a contiguous torch.* tensor on the GPU"):
        CALLS[call](arguments())


@pytest.mark.parametrize("call,name,value", [
    ("forward", "array", torch.zeros(M + 1)), ("forward", "out", torch.zeros(B, F, D + 1)), ("forward", "offsets", torch.zeros(B * F, dtype=torch.int64)),
    ("bf16", "array", torch.zeros(M + 1)), ("backward", "grad", torch.zeros(M - 1)), ("backward", "grad_out", torch.zeros(B, F)),
    ("noalloc", "grad_out", torch.zeros(1)), ("adagrad", "state", torch.zeros(2)), ("sgd", "grad", torch.zeros(2)),
    ("fused", "state", torch.zeros(M + 2)), ("fused_sgd", "grad_out", torch.zeros(3)), ("mixed", "array", torch.zeros(3)),
    ("mixed_backward", "dims", [16, 8, 8]), ("mixed_fused", "offsets", torch.zeros(2, dtype=torch.int64))])
def test_wrong_lengths_are_refused(call, name, value):
    a = arguments()
    a[name] = value
    with pytest.raises(ValueError):
        CALLS[call](a)


@pytest.mark.parametrize("call,name,value", [("forward", "h", 3), ("forward", "array", None), ("backward", "ids", [1, 2]), ("sgd", "array", "x"),
                                             ("adagrad", "state", None), ("fused", "state", None), ("mixed", "dims", 5),
                                             ("forward", "options", torch.zeros(1))])
def test_wrong_kinds_are_refused(call, name, value):
    a = arguments()
    a[name] = value
    with pytest.raises((TypeError, BufferError)):
        CALLS[call](a)
