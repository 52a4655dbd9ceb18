"""The binding's workspace cache (no GPU): the workspace of a captured call, which the graph's replays write,
outlives a larger one on the same stream until the cache is cleared."""
import types
import weakref

import numpy as np

from paper_1002_1050_amd import _binding as B


class Buf(np.ndarray):
    def numel(self):
        return self.size


def fake_torch(capturing):
    cuda = types.SimpleNamespace(is_current_stream_capturing=lambda: capturing[0])
    return types.SimpleNamespace(cuda=cuda, uint8=np.uint8,
                                 empty=lambda n, dtype, device: np.empty(n, dtype).view(Buf))


def test_captured_workspace_is_kept():
    capturing = [False]
    torch, device, stream = fake_torch(capturing), types.SimpleNamespace(index=0), types.SimpleNamespace(value=7)
    cache = B._Workspace()
    first = weakref.ref(cache.get(torch, device, stream, 1000))
    assert cache.get(torch, device, stream, 500) is first()          # grow-only
    second = weakref.ref(cache.get(torch, device, stream, 2000))
    assert first() is None                                           # nobody's any more
    capturing[0] = True
    assert cache.get(torch, device, stream, 1500) is second()        # a graph holds its address now
    capturing[0] = False
    third = weakref.ref(cache.get(torch, device, stream, 4000))
    assert second() is not None and third() is not second()
    assert cache.get(torch, device, stream, 4000) is third()
    cache.clear()
    assert second() is None and third() is None
