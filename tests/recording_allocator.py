"""An allocator over torch that notes what the library asks of it, and has only so much to give."""
import torch


class RecordingAllocator:
    """live, peak: device bytes handed out, now and at most; requested: their sum over all requests.  total_bytes: a request that
    would take `live` above it is refused (NULL to the library), as an allocator that has run out would."""

    def __init__(self, rg, total_bytes=None):
        self.blocks, self.live, self.peak, self.requested, self.n_refused = {}, 0, 0, 0, 0

        def alloc(nbytes, kind, _ctx):
            n = int(nbytes)
            if kind == 1 and total_bytes is not None and self.live + n > total_bytes:
                self.n_refused += 1
                return None
            t = torch.empty(n, dtype=torch.uint8, device="cuda") if kind == 1 else torch.empty(n, dtype=torch.uint8, pin_memory=True)
            self.blocks[t.data_ptr()] = (t, n if kind == 1 else 0)
            if kind == 1:
                self.live += n
                self.peak = max(self.peak, self.live)
                self.requested += n
            return t.data_ptr()

        def free(p, _kind, _ctx):
            self.live -= self.blocks.pop(p)[1]

        self._fns = rg.ALLOC_FN(alloc), rg.FREE_FN(free)
        self.struct = rg.rg_allocator(*self._fns, None)
