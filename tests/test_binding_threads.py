"""What a Config keeps is the same object for every thread, also when several ask for it first at once."""
import ctypes
import threading

from paper_2510_06175_amd import binding as vb


def test_kept_address_is_of_the_kept_struct(monkeypatch):
    """A second thread asks for the struct's address while the first is still building the struct: the address
    that is kept for the native calls must be that of the struct that is kept (the other one is freed)."""
    cfg, build, calls = vb.Config(128, 32, 8, 4, 4), vb.Config.c, []

    def interrupted(self):
        struct = build(self)
        calls.append(struct)
        if len(calls) == 1:
            other = threading.Thread(target=lambda: self._p)
            other.start()
            other.join()
        return struct

    monkeypatch.setattr(vb.Config, "c", interrupted)
    mine = cfg._c
    assert len(calls) == 2
    assert cfg._c is mine
    assert cfg._p == ctypes.addressof(cfg._c)
