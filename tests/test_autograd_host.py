"""The host side of the autograd glue, on the CPU."""
import types

import torch

from paper_2403_08148_amd import autograd as G


def test_type_pair_weights_whatever_the_default_device():
    """The factors kept with an engine are made on the host and copied to the
    engine's device, also where a program has set another default device."""
    engine = types.SimpleNamespace(device=torch.device("cpu"))
    with torch.device("meta"):
        w = G._sym_weights(engine, 3)
    assert w.device.type == "cpu"
    assert torch.equal(w, torch.where(torch.eye(3) > 0, 1.0, 0.5).double())
    assert G._sym_weights(engine, 3) is w
