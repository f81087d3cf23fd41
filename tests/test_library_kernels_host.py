"""CPU checks of the compiled kernels' registers, from the metadata of the library built here: the
persistent one-launch kernels keep several tiles' code in one loop, where the compiler tends to hold every
tile's constants in registers and leaves the chip half empty."""
import os
import re
import struct
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, 'paper_2608_14123_amd', 'libdgfas.so')
READELF = '/opt/rocm/llvm/bin/llvm-readelf'


@pytest.fixture(scope='module')
def vgprs():
    """Vector registers per kernel (demangled up to its argument list)."""
    if not os.path.exists(LIB):
        pytest.fail('libdgfas.so is not built (run __graft_entry__.build())')
    blob, found = open(LIB, 'rb').read(), {}
    at = blob.find(b'\x7fELF', 1)
    while at >= 0:
        size = 4
        if struct.unpack_from('<H', blob, at + 18)[0] == 224:    # an AMDGPU code object: ends with its section table
            size = struct.unpack_from('<Q', blob, at + 40)[0]
            size += struct.unpack_from('<H', blob, at + 58)[0] * struct.unpack_from('<H', blob, at + 60)[0]
            with tempfile.NamedTemporaryFile() as f:
                f.write(blob[at:at + size])
                f.flush()
                notes = subprocess.run([READELF, '--notes', f.name], capture_output=True, text=True, check=True).stdout
            for k in re.split(r'\n\s+- \.agpr_count:', notes)[1:]:
                found[re.search(r'\.name:\s+(\S+)', k)[1]] = int(re.search(r'\.vgpr_count:\s+(\d+)', k)[1])
        at = blob.find(b'\x7fELF', at + size)
    names = subprocess.run(['c++filt'], input='\n'.join(found), capture_output=True, text=True, check=True).stdout
    return {n.replace('void ', '').replace('dgfas::', '').split('(')[0]: v for n, v in zip(names.split('\n'), found.values())}


@pytest.mark.parametrize('n', [6, 7, 8, 9])
@pytest.mark.parametrize('t,waves', [('double', 6), ('float', 8)])
def test_persistent_subdomain_solve_occupancy(vgprs, n, t, waves):
    # 512 registers per SIMD lane, in units of 8
    used = vgprs['schwarz_batched_kernel<%d, %s, true>' % (n, t)]
    assert 512 // ((used + 7) // 8 * 8) >= waves, used
