"""A factorization that fills the device: where the W of several waiting panels does not fit
beside the factors, it keeps one panel's, with the same results."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1908_06043_amd import _lib

pytestmark = pytest.mark.gpu


def test_factorization_with_room_for_one_panel(gpu_lib):
    n, S = 8192, 48       # W of six panels: 1.2 GB, of one 0.2; 0.2 besides
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    A = torch.randn((n, n), generator=g, dtype=torch.float64, device="cuda")
    A = (0.5 * (A + A.T)).contiguous()
    # mostly accepted without pivoting, so that panels wait for one another
    A.diagonal()[: n - 700] += 300.0
    B = torch.eye(n, dtype=torch.float64, device="cuda")
    sig = np.linspace(-20.0, 20.0, S)
    ref = gpu_lib.ldlt_factor_multi(A, B, sig)
    lib = _lib.load()
    h = C.c_void_p()
    assert lib.sislice_create(C.byref(h), torch.cuda.current_device(), None) == 0
    LD = [torch.empty((n, n), dtype=torch.float64, device="cuda") for _ in range(S)]
    ip = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(S)]
    inert = np.zeros(3 * S, dtype=np.int64)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    fill = torch.empty((free - (1050 << 20)) // 8, dtype=torch.float64, device="cuda")
    try:
        ptrs = lambda ts: (C.c_void_p * S)(*[t.data_ptr() for t in ts])
        print(f"free {torch.cuda.mem_get_info()[0] >> 20} MiB", flush=True)
        for _ in range(2):
            st = lib.sislice_ldlt_factor_multi(h, n, A.data_ptr(), n, B.data_ptr(), n, S,
                                               sig.ctypes.data_as(_lib.c_double_p), ptrs(LD), n, ptrs(ip),
                                               inert.ctypes.data_as(_lib.c_int64_p))
            assert st == 0
    finally:
        del fill
        lib.sislice_destroy(h)
        torch.cuda.empty_cache()
    for s in range(S):
        assert ref[s].inertia == tuple(int(x) for x in inert[3 * s:3 * s + 3])
        assert torch.equal(ref[s].ipiv, ip[s])
    for s in (0, 20, S - 1):
        assert torch.equal(torch.tril(ref[s].LD), torch.tril(LD[s].t()))
