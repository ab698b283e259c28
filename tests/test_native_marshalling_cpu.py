"""What the native marshalling hands to the C entry points and what it refuses, without a GPU: the entry points are replaced by
functions that record their arguments and return a status."""
import pytest
import torch

import paper_2605_21072_amd as q
from paper_2605_21072_amd import binding


@pytest.fixture
def no_stream(monkeypatch):
    """The current stream's handle without a device to have one."""
    if not q.lib_path().exists():
        from paper_2605_21072_amd import build
        build.build()
    q.load_library()
    monkeypatch.setattr(binding, "_stream", lambda stream: 0)


def test_a_static_scale_that_is_no_number_is_refused(no_stream):
    X = torch.zeros((4, 128))
    for scale in (None, "0.1", [0.1]):
        with pytest.raises(TypeError):
            q.quant_act_static(X, None, 0, scale)
