"""Calls without a stream argument go to torch's current stream, whichever it is and whichever thread asks."""
import threading

import pytest
import torch

import paper_2501_18512_amd as sdl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["default", "side", "thread"])
def test_default_stream_is_the_current_one(where):
    torch.cuda.current_stream()
    side, got = torch.cuda.Stream(), []

    def ask():
        got.append((sdl._stream(None), torch.cuda.current_stream().cuda_stream))

    if where == "side":
        with torch.cuda.stream(side):
            ask()
        assert got[0][0] == side.cuda_stream
    elif where == "thread":
        with torch.cuda.stream(side):
            t = threading.Thread(target=ask)      # a new thread starts on the default stream
            t.start()
            t.join()
        assert got[0][0] != side.cuda_stream
    else:
        ask()
    assert got[0][0] == got[0][1]
    # explicit streams are passed on as they are
    assert sdl._stream(side) == side.cuda_stream and sdl._stream(1234) == 1234
