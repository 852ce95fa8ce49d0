"""Cases of test_host_paths_cpu.py, each run in a process of its own on the
HIP runtime in host memory (host_hip.py)."""
import ctypes as C
import struct

import numpy as np


def _part_sums(launch):
    """(first byte, bytes) of every region of partial sums that k_sum_parts reads."""
    raw = bytes(launch.arg)
    n_jobs = struct.unpack_from("<i", raw, 12 * 32)[0]
    out = []
    for k in range(n_jobs):
        src, _, rows, cols, stride, _ = struct.unpack_from("<QQiiii", raw, 32 * k)
        out.append((src, 4 * ((rows - 1) * stride + cols)))
    return out


def gradient_parts(hh, gsp):
    """The partial sums of every batch fit the buffer that any larger batch
    reserved (a training set's last batch is a short one)."""
    ctx = gsp.Context(0)
    top = 8192
    host = np.zeros(1 << 20, np.float32)
    loss = C.c_float()

    def call(net, n):
        hh.clear()
        rc = gsp.lib().gsp_cnn_gradients(net.h, 4096, 4096, n, host.ctypes.data_as(C.c_void_p), C.byref(loss), None)
        assert rc == gsp.GSP_OK, (n, rc)
        (sums,) = hh.launches("k_sum_parts")
        regions = _part_sums(sums)
        base = min(p for p, _ in regions)
        return base, max(p + b for p, b in regions) - base

    big = gsp.Cnn(ctx, seed=1)
    call(big, top)
    need = np.array([0] + [call(big, n)[1] for n in range(1, top + 1)])
    big.close()
    for r in (1, 171, 204, 205, 256, 384, 512, 1000, 2592, top):
        net = gsp.Cnn(ctx, seed=1)
        base, _ = call(net, r)
        room = hh.room(base)
        assert room >= need[:r + 1].max(), f"{r} images reserve {room} bytes, {need[:r + 1].argmax()} take {need[:r + 1].max()}"
        net.close()
