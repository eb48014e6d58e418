"""Number of kernels that a call enqueues, from a HIP graph captured of it."""
import ctypes

import torch


def _hip():
    with open("/proc/self/maps") as f:
        path = next(ln.split()[-1] for ln in f if "libamdhip64.so" in ln)
    return ctypes.CDLL(path)


def count(fn, set_stream) -> int:
    """Nodes of the graph captured of fn(); set_stream(handle) puts the
    library's context on the capturing stream (and back)."""
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        set_stream(s.cuda_stream)
        fn()  # (once outside the capture)
        s.synchronize()
        g.capture_begin()
        fn()
        g.capture_end()
        n = ctypes.c_size_t(0)
        assert _hip().hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    torch.cuda.current_stream().wait_stream(s)
    set_stream(torch.cuda.current_stream().cuda_stream)
    return n.value
