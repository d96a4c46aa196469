"""Which plan a search call takes (test helper): the workspace it insists on, and the tile kernels it launches."""
import ctypes
import re
import warnings

import torch

from paper_2507_21433_amd import binding as rc

FAKE = ctypes.c_void_p(0x1000)      # never dereferenced: a call without a workspace is refused before anything is launched


def descs(L, T, H, P, Q):
    return [rc.KvDesc(L, T, H, 128, 0, n * T * H * 128) for n in (Q, P)]


def _said(lib):
    return int(re.search(rb"workspace of (\d+) bytes needed", lib.rc_last_error()).group(1))


def needed(lib, mode, L, T, H, P, Q):
    """What rc_match_blocks says it needs."""
    q, p = descs(L, T, H, P, Q)
    assert lib.rc_match_blocks(ctypes.byref(q), ctypes.byref(p), mode, FAKE, FAKE, Q, FAKE, FAKE, FAKE, FAKE, P, FAKE, FAKE, None,
                               0.9, FAKE, FAKE, FAKE, None, None, 0, None) == 3
    return _said(lib)


def size(lib, mode, L, T, H, P, Q):
    return lib.rc_match_workspace_size(ctypes.byref(descs(L, T, H, P, Q)[0]), mode, Q, P)


def mean_needed(lib, L, T, H, P, Q):
    """What rc_match_blocks_layer_mean says it needs."""
    q, p = descs(L, T, H, P, Q)
    assert lib.rc_match_blocks_layer_mean(ctypes.byref(q), ctypes.byref(p), FAKE, FAKE, Q, FAKE, FAKE, FAKE, FAKE, P, FAKE, FAKE, None,
                                          0.5, FAKE, FAKE, FAKE, None, None, 0, None) == 3
    return _said(lib)


def mean_size(lib, L, T, H, P, Q):
    return lib.rc_layer_mean_workspace_size(ctypes.byref(descs(L, T, H, P, Q)[0]), Q, P)


def whole_tiles(L, P, Q):
    """Need of whole tiles: 16 bytes per (layer, pool tile of 256, query), then the tile schedule: 520 words of 128 bytes,
    one claim word per tile of the launch (rounded up to rounds of 256) and 512 more."""
    npt, nqt = -(-P // 256), -(-Q // 256)
    return L * npt * Q * 16 + 4 * (520 * 32 + -(-L * npt * nqt // 256) * 256 + 512)


def whole_tiles_workspace(w):
    """A workspace that has room for whole tiles with pool tiles of 256 rows and for nothing else."""
    n = needed(rc.lib(), w.mode, w.L, w.T, w.H, w.P, w.Q)
    assert n == whole_tiles(w.L, w.P, w.Q), "a shape whose need is that of shares"
    return torch.empty(n, dtype=torch.uint8, device="cuda:0")


def kernel_names(call):
    """Names of the kernels that call() launches, [] where no kernel trace is to be had.  The profiler can lose events, all of
    them in a trace of a few microseconds: a trace without any is taken again, of more calls."""
    from torch.profiler import ProfilerActivity, profile
    for times in (3, 12, 48):
        with warnings.catch_warnings():
            warnings.simplefilter("ignore")
            with profile(activities=[ProfilerActivity.CUDA]) as p:
                for _ in range(times):
                    call()
                torch.cuda.synchronize()
        names = [e.name for e in p.events()]
        if any("rc::" in n for n in names):
            return names
    return []


def tile_kernels(call):
    """{(pool rows, columns, mode)} of the tile kernels that call() launches; None where no kernel trace is to be had."""
    names = kernel_names(call)
    if not names:
        return None
    found = [re.search(r"match_(?:tile|shape)_kernel<\w+, (\d+), (\d+), (\d)", n) for n in names]
    return {tuple(int(x) for x in m.groups()) for m in found if m}


def assert_tiles(call, *want):
    for _ in range(3):      # a trace that has lost some of the wanted kernels is taken again; one that has others is not
        got = tile_kernels(call)
        if got is None or not got < set(want):
            break
    assert got in (None, set(want)), f"tile kernels {sorted(got)}, the test is about {want}"
