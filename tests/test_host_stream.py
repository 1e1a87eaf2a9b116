"""The stream that a launch takes, without a GPU: torch's raw-stream call
where the build has it, else the public Stream object."""
import types

import pytest

from paper_2510_12897_amd import opf


@pytest.mark.parametrize("names,want", [((), 7), (("_cuda_getDevice",), 7), (("_cuda_getCurrentRawStream",), 7),
                                        (("_cuda_getDevice", "_cuda_getCurrentRawStream"), 5)])
@pytest.mark.parametrize("initialized", [True, False])
def test_current_stream_without_the_private_names(monkeypatch, names, want, initialized):
    private = {"_cuda_getDevice": lambda: 0, "_cuda_getCurrentRawStream": lambda dev: 5}
    fake = types.SimpleNamespace(
        _C=types.SimpleNamespace(**{k: private[k] for k in names}),
        cuda=types.SimpleNamespace(is_initialized=lambda: initialized,
                                   current_stream=lambda: types.SimpleNamespace(cuda_stream=7)))
    monkeypatch.setattr(opf, "_torch_module", fake)
    assert opf._stream() == (want if initialized else 7)
