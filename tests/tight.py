"""A context whose arena has exactly the size asked for, with a guard of known
bytes behind it."""
import ctypes

import torch

import paper_1104_3830_amd as sk

GUARD = 4 << 20
FILL = 0xA5


class TightContext(sk.Context):
    def _alloc(self, nbytes):
        assert self._ptr is None, "the size given does for every call"
        self.buf = torch.full((nbytes + GUARD,), FILL, dtype=torch.uint8, device=self.device)
        self.arena = self.buf[:nbytes]
        ptr = ctypes.c_void_p()
        st = sk.lib().sk_create(ctypes.byref(ptr), self.device.index or 0, ctypes.c_void_p(self.stream.cuda_stream),
                                ctypes.c_void_p(self.arena.data_ptr()), nbytes)
        assert st == sk.SK_OK
        self._ptr = ptr

    def ensure_arena(self, nbytes):
        """Calls run in the arena there is, whatever the sizing functions say."""

    def guard_untouched(self):
        return bool((self.buf[self.arena.numel():] == FILL).all())
