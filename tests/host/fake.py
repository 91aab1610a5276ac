"""The library over the recording runtime of fake_hip.cpp: loaded in a process of its own, before anything else that
links the real one.  `python fake.py <libfake_hip.so> <function>` runs a function of test_host_routes.py."""
import ctypes
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
FIELDS = ("grid", "threads", "stream", "tiles", "merges", "waves", "scratch", "counters", "list")


class Fake:
    def __init__(self, path):
        self.lib = ctypes.CDLL(path, mode=ctypes.RTLD_GLOBAL)
        for name in ("fake_live", "fake_count"):
            getattr(self.lib, name).restype = ctypes.c_int64
        self.lib.fake_name.restype = ctypes.c_char_p
        self.lib.fake_limit_device_memory.argtypes = [ctypes.c_int64]

    def limit(self, more):
        """At most `more` further bytes of device memory (None: no limit)."""
        self.lib.fake_limit_device_memory(-1 if more is None else more)

    def live(self):
        return self.lib.fake_live()

    def count(self, what):
        return self.lib.fake_count(what.encode())

    def forget(self):
        self.lib.fake_forget()

    def _rows(self, call, i, n, width):
        out = (ctypes.c_int64 * (n * width))()
        call(i, out)
        return [tuple(out[k * width:(k + 1) * width]) for k in range(n)]

    def launches(self, part=""):
        """Launches of kernels whose name has `part` in it, each a dict."""
        found = []
        for i in range(self.lib.fake_launches()):
            name = self.lib.fake_name(i).decode()
            if part in name:
                d = dict(zip(FIELDS, self._rows(self.lib.fake_launch, i, 1, len(FIELDS))[0]), name=name)
                d["units"] = self._rows(self.lib.fake_tiles, i, d["tiles"], 8)
                d["merged"] = self._rows(self.lib.fake_merges, i, d["merges"], 5) if "merge" in name else []
                d["named"] = self._rows(self.lib.fake_units, i, self.lib.fake_unit_count(i), 2)
                d["slots"] = [u[0] for u in self._rows(self.lib.fake_slots, i, d["tiles"], 1)] if d["merges"] and d["tiles"] else []
                d["places"] = self._rows(self.lib.fake_places, i, d["merges"], 2) if "merge" in name else []
                found.append(d)
        return found


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    fake = Fake(sys.argv[1])                      # before libpbkv.so
    from tests import test_host_routes
    getattr(test_host_routes, sys.argv[2])(fake, *sys.argv[3:])
    print("clean")
