"""The layer's host side (no GPU): what it hands to the library follows the tensors that it holds."""
import copy
import pickle

import torch

import paper_2605_27003_amd as svdq


def test_descriptor_follows_the_layer():
    qw, sw = torch.zeros((128, 32), dtype=torch.uint8), torch.ones((1, 128))
    lin = svdq.W4A4Linear(torch.ones(64), None, None, qw, sw, torch.zeros(128))
    lin._descriptor(0)
    for other in (copy.copy(lin), copy.deepcopy(lin), pickle.loads(pickle.dumps(lin))):
        other.bias = torch.ones(128)
        other._descriptor(0)
        assert other._layer.bias == other.bias.data_ptr() and other._layer.qw == other.qw.data_ptr()
    lin.bias = None
    lin._descriptor(16)
    assert lin._layer.bias is None and lin._layer.r == 16
