"""Scenarios of tests/test_host_runtime.py: each runs in a process of its own, as
``python -m tests.host_runtime.scenarios NAME FAKE_LIBRARY``, with the library's HIP calls going to fake_hip.cpp."""
import ctypes
import sys

import numpy as np

import paper_2512_15550_amd as ck

OK, EINVAL, EHIP, EUNSUPPORTED = 0, -1, -3, -4


class Host:
    def __init__(self, fake_path):
        self.fake = ctypes.CDLL(fake_path, mode=ctypes.RTLD_GLOBAL)
        self.fake.fake_live_bytes.restype = ctypes.c_size_t
        self.lib = ck.load_library()

    def device(self, d):
        assert self.fake.hipSetDevice(d) == 0

    def current(self):
        d = ctypes.c_int(-1)
        self.fake.hipGetDevice(ctypes.byref(d))
        return d.value

    def load(self, s=4096, C=64, rho=256, h=8, g=2, probe=8, top_k=256, batch=1, expect=OK):
        p = ck.Params(batch=batch, n_q_heads=h, n_kv_heads=g, dtype=ck.BF16, n_centroids=C, list_len=rho, n_probe=probe, top_k=top_k).c()
        lens = np.full(batch, s, np.int32)
        cen = np.random.RandomState(s).randint(0, 1 << 16, (batch, h, C, 128)).astype(np.uint16)
        lists = np.tile(np.arange(rho, dtype=np.int32), (batch, g, C, 1))
        out = ctypes.c_void_p()
        rc = self.lib.ctkvr_index_load(ctypes.byref(p), lens.ctypes.data, cen.ctypes.data, lists.ctypes.data, None, ctypes.byref(out))
        assert rc == expect, (rc, ck.ctkvr_last_error())
        return out.value, cen, lists

    def info(self, ix):
        i = ck.binding._CInfo()
        assert self.lib.ctkvr_index_info(ix, ctypes.byref(i)) == OK
        return i


def refused_wait(x):
    """An index freed while the device cannot be waited for (a stream is being captured): its memory goes to no other
    index, and is not freed, until a later wait has succeeded."""
    a, _, _ = x.load()
    n, held = x.fake.fake_mallocs(), x.fake.fake_live_bytes(0)
    x.fake.fake_refuse_syncs(1, 0)
    x.lib.ctkvr_free(a)
    assert x.fake.fake_live_bytes(0) == held
    assert x.fake.hipGetLastError() == 0, "the refused wait is left for the next check of a launch"
    b, _, _ = x.load()                       # still refused: memory of its own
    assert x.fake.fake_mallocs() == n + 1, "memory that may still be in use was handed to another index"
    assert x.lib.ctkvr_release_scratch() == OK and x.fake.fake_live_bytes(0) == 2 * held
    x.fake.fake_refuse_syncs(0, 0)
    s = x.fake.fake_syncs(0)
    c, _, _ = x.load()                       # waited for now: the first index's memory
    assert x.fake.fake_syncs(0) > s and x.fake.fake_mallocs() == n + 1
    x.lib.ctkvr_free(b)
    x.lib.ctkvr_free(c)
    assert x.lib.ctkvr_release_scratch() == OK and x.fake.fake_live_bytes(0) == 0


def refused_wait_released(x):
    """... and ctkvr_release_scratch frees it once the wait succeeds."""
    a, _, _ = x.load()
    x.fake.fake_refuse_syncs(1, 0)
    x.lib.ctkvr_free(a)
    x.fake.fake_refuse_syncs(0, 0)
    assert x.lib.ctkvr_release_scratch() == OK and x.fake.fake_live_bytes(0) == 0


def refused_build(x):
    """A build whose stream cannot be waited for fails, and its scratch is set aside like the memory of an index."""
    p = ck.Params(batch=1, n_q_heads=8, n_kv_heads=2, dtype=ck.BF16, n_centroids=64, list_len=256, n_probe=8, top_k=256).c()
    lens, cu, out = np.array([4096], np.int32), np.array([0, 64], np.int32), ctypes.c_void_p()
    ptr = ctypes.c_void_p(4096)              # (kernels do nothing here)

    def build():
        return x.lib.ctkvr_build_index(ctypes.byref(p), ptr, cu.ctypes.data, 1, ptr, ptr, 256, lens.ctypes.data, None, None,
                                       ctypes.byref(out))

    x.fake.fake_refuse_syncs(1, 1)
    assert build() == EHIP
    n, held = x.fake.fake_mallocs(), x.fake.fake_live_bytes(0)
    assert n == 2 and x.fake.fake_frees() == 0
    assert build() == EHIP and x.fake.fake_mallocs() == 2 * n, "scratch that may still be in use was handed to another build"
    x.fake.fake_refuse_syncs(0, 0)
    assert build() == OK and x.fake.fake_mallocs() == 2 * n
    x.lib.ctkvr_free(out.value)
    assert x.lib.ctkvr_release_scratch() == OK and x.fake.fake_live_bytes(0) == 0


def refused_copy(x):
    """A load whose copies cannot be waited for fails, and the pinned memory they go through serves no other copy, and is not
    freed, until the device has been waited for."""
    a, cen, _ = x.load(C=512)                # (large enough for the pinned memory)
    assert x.fake.fake_pinned() == 1 and x.fake.fake_records() > 0
    x.fake.fake_refuse_syncs(1, 1)
    x.load(C=512, expect=EHIP)
    n = x.fake.fake_records()
    got = np.empty_like(cen)
    x.fake.fake_refuse_syncs(1, 0)
    x.load(C=512)
    assert x.fake.fake_records() == n, "pinned memory that may still be in use took part in another copy"
    assert x.lib.ctkvr_release_scratch() == OK and x.fake.fake_pinned() == 1
    x.fake.fake_refuse_syncs(0, 0)
    assert x.lib.ctkvr_index_centroids(a, got.ctypes.data) == OK and np.array_equal(got, cen)
    assert x.fake.fake_records() > n
    assert x.lib.ctkvr_release_scratch() == OK and x.fake.fake_pinned() == 0


def other_device(x):
    """The inspection calls work on the index's device whichever is current, wait for that one, and leave the current one."""
    x.device(1)
    a, cen, lists = x.load(C=512)
    assert x.lib.ctkvr_release_scratch() == OK      # (the pinned memory is made again, now with device 0 current)
    x.device(0)
    got_c, got_l, last = np.empty_like(cen), np.empty_like(lists), np.empty((2, 8 * 256), np.int32)
    err = ctypes.c_int32(0)
    for call in (lambda: x.lib.ctkvr_index_centroids(a, got_c.ctypes.data), lambda: x.lib.ctkvr_index_lists(a, got_l.ctypes.data),
                 lambda: x.lib.ctkvr_index_last_candidates(a, last.ctypes.data), lambda: x.lib.ctkvr_profile_phases(a, 0, None),
                 lambda: x.lib.ctkvr_profile_enable(a, 2), lambda: x.lib.ctkvr_profile_collect(a, last.ctypes.data, 2, ctypes.byref(err))):
        n0, n1 = x.fake.fake_syncs(0), x.fake.fake_syncs(1)
        assert call() == OK, ck.ctkvr_last_error()
        assert x.current() == 0 and x.fake.fake_syncs(0) == n0 and x.fake.fake_syncs(1) > n1
    n1 = x.fake.fake_syncs(1)
    x.lib.ctkvr_index_check(a)                      # (its word reads as an error: no kernel has cleared it)
    assert x.current() == 0 and x.fake.fake_syncs(1) > n1
    assert np.array_equal(got_c, cen) and np.array_equal(got_l, lists)
    x.device(1)
    b, _, _ = x.load(C=512)                         # the pinned memory as the export left it
    assert x.lib.ctkvr_index_centroids(b, got_c.ctypes.data) == OK
    x.device(0)
    x.lib.ctkvr_free(a)
    assert x.current() == 0


def path_of_other_device(x):
    """Choosing the single launch raises the kernel's shared-memory limit on the index's device."""
    x.device(1)
    a, _, _ = x.load()
    x.device(0)
    n = x.fake.fake_attr_calls()
    assert x.lib.ctkvr_index_set_decode_path(a, ck.PATH_FUSED) == OK
    assert x.fake.fake_attr_calls() > n and x.fake.fake_attr_device() == 1 and x.current() == 0


def memory_held(x):
    """ctkvr_index_info names all that an index holds; kept memory makes that at most a quarter more than the index needs, and
    the boundaries between an index's parts at most a fifth."""
    big = dict(s=32768, C=512, rho=1024, h=32, g=8, probe=32, top_k=1024)
    own = {}
    for name, over in (("big", {}), ("near", dict(C=460)), ("less", dict(C=300)), ("small", dict(s=4096, C=64, rho=256, h=8, g=2, probe=8, top_k=256))):
        a, _, _ = x.load(**{**big, **over})
        own[name] = x.info(a).device_bytes
        assert own[name] == x.fake.fake_live_bytes(0)
        x.lib.ctkvr_free(a)
        assert x.lib.ctkvr_release_scratch() == OK
    a, _, _ = x.load(**big)
    x.lib.ctkvr_free(a)
    n = x.fake.fake_mallocs()
    a, _, _ = x.load(**{**big, **dict(C=460)})
    assert x.fake.fake_mallocs() == n and x.info(a).device_bytes == own["big"] <= 1.25 * own["near"]
    x.lib.ctkvr_free(a)
    a, _, _ = x.load(**{**big, **dict(C=300)})
    assert x.info(a).device_bytes == own["less"], "an index holds far more than it needs"
    # the 4K index: centroids, their norms and lists (0.26 MiB), what a step writes (1.7 MiB)
    assert own["small"] <= 5 << 19


def static_scratch_holds(x):
    """The static scratch array takes what the step's buffers need with a cache line per unit for the words that atomics update: 1104
    units of the smallest size need 31.8 MiB without those lines, 32.2 with them; what needs more than 32 without them is refused, also where
    it would fit the room that is there for the lines."""
    ptr = ctypes.c_void_p(4096)              # (kernels do nothing here)
    small = dict(s=64, C=4, rho=16, h=8, g=8, probe=4, top_k=16)
    long = dict(s=100000, C=64, rho=2048, h=8, g=2, probe=64, top_k=2048, batch=4)
    for geo, rc in ((dict(small, batch=138), OK), (dict(small, batch=142), EUNSUPPORTED), (long, EUNSUPPORTED)):
        a, _, _ = x.load(**geo)
        assert x.lib.ctkvr_decode_step_static(a, ptr, ptr, ptr, ptr, -(-geo["s"] // 16), ptr, None, None, None, None, None) == rc, ck.ctkvr_last_error()
        x.lib.ctkvr_free(a)


SCENARIOS = {f.__name__: f for f in (refused_wait, refused_wait_released, refused_build, refused_copy, other_device, path_of_other_device, memory_held,
                                     static_scratch_holds)}

if __name__ == "__main__":
    SCENARIOS[sys.argv[1]](Host(sys.argv[2]))
    print("ok")
