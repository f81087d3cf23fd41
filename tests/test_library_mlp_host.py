"""The network's workspace when memory runs out, on the CPU: csrc/mlp.hip built with g++ through
tests/mlp_alloc_shim.cpp, whose stand-ins for the HIP runtime let one allocation after another fail."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OK, ENOMEM = 0, -2
IN, H, OUT, SMALL, LARGE = 12, 8, 5, 4, 64


@pytest.fixture(scope='module')
def shim(tmp_path_factory):
    so = str(tmp_path_factory.mktemp('mlp') / 'mlp_alloc.so')
    subprocess.run(['g++', '-std=c++17', '-O1', '-shared', '-fPIC', '-D__HIP_PLATFORM_AMD__', '-I/opt/rocm/include',
                    '-Wno-unused-result', '-x', 'c++', os.path.join(ROOT, 'tests', 'mlp_alloc_shim.cpp'), '-o', so], check=True)
    lib = ctypes.CDLL(so)
    lib.shim_alloc.restype = ctypes.c_void_p
    lib.shim_alloc.argtypes = [ctypes.c_size_t]
    lib.shim_free.argtypes = [ctypes.c_void_p]
    V, I = ctypes.c_void_p, ctypes.c_int32
    lib.dgfas_mlp_create.argtypes = [I, I, I, ctypes.c_uint64, V, ctypes.POINTER(V)]
    lib.dgfas_mlp_forward.argtypes = [V, V, I, V]
    lib.dgfas_mlp_gradient.argtypes = [V, V, V, I, V, ctypes.POINTER(ctypes.c_double)]
    lib.dgfas_mlp_destroy.argtypes = [V]
    return lib


# a larger batch allocates nine buffers, its gradient one more for the outputs
@pytest.mark.parametrize('call,allocations', [('forward', 9), ('gradient', 10)])
@pytest.mark.parametrize('warm', [False, True])
def test_failed_growth_leaves_a_usable_network(shim, call, allocations, warm):
    for k in range(allocations + 1):
        net = ctypes.c_void_p()
        assert shim.dgfas_mlp_create(IN, H, OUT, 5, None, ctypes.byref(net)) == OK
        X, T, Y = (shim.shim_alloc(4 * LARGE * n) for n in (IN, OUT, OUT))

        def run(rows):
            if call == 'forward':
                return shim.dgfas_mlp_forward(net, X, rows, Y)
            return shim.dgfas_mlp_gradient(net, X, T, rows, None, ctypes.byref(ctypes.c_double()))

        if warm:
            assert run(SMALL) == OK
        shim.shim_fail_at(k)
        assert run(LARGE) == (ENOMEM if k < allocations else OK)
        shim.shim_fail_at(-1)
        assert shim.shim_faults() == 0
        # smaller and larger calls after the failure, and the end of the network
        for rows in (SMALL, LARGE, SMALL):
            assert run(rows) == OK
            assert shim.shim_faults() == 0, (k, rows)
        shim.dgfas_mlp_destroy(net)
        for p in (X, T, Y):
            shim.shim_free(p)
        assert shim.shim_faults() == 0 and shim.shim_live() == 0, k
