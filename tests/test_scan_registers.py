"""Registers of the scan and L1 base kernels, from the metadata of the built
library.

Under L2 and L1 a scan kernel computes its LUT from the residuals; the copy of
a query's inner-product table belongs to kernels of its own, so its registers
cost these searches no wavefronts in flight.  A SIMD has 512 vector registers
per lane, handed out in steps of 8: 72 of them leave seven waves, 96 five.  L1's pair bases run on the VALU,
without the matrix fragments of the other builds' bases.  The mixed-class scans
hold the widest of their lane classes' bodies without, or nearly without,
scratch memory.
"""
import os
import struct

import pytest

import paper_2606_07156_amd as amp

msgpack = pytest.importorskip("msgpack")
LIB = os.path.join(os.path.dirname(os.path.abspath(amp.__file__)), "libamp.so")
EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def _kernels():
    """{mangled name: metadata} of every kernel in the library's code objects."""
    b, out, at = open(LIB, "rb").read(), {}, 0
    while (at := b.find(b"\x7fELF", at + 1)) >= 0:
        if struct.unpack_from("<H", b, at + 18)[0] != EM_AMDGPU:
            continue
        shoff = struct.unpack_from("<Q", b, at + 40)[0]
        size, count = struct.unpack_from("<HH", b, at + 58)
        for s in range(at + shoff, at + shoff + size * count, size):
            if struct.unpack_from("<I", b, s + 4)[0] != SHT_NOTE:
                continue
            off, n = struct.unpack_from("<QQ", b, s + 24)
            p, end = at + off, at + off + n
            while p < end:
                ns, ds, kind = struct.unpack_from("<III", b, p)
                d = p + 12 + (ns + 3 & ~3)
                if kind == NT_AMDGPU_METADATA:
                    for k in msgpack.unpackb(b[d:d + ds])["amdhsa.kernels"]:
                        out[k[".name"]] = k
                p = d + (ds + 3 & ~3)
    return out


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    return _kernels()


# k_scan<0 (FP32), subspaces (0: generic), phase, 1 (no table copy), 0, threads>
@pytest.mark.parametrize("phase", [1, 2, 3])
@pytest.mark.parametrize("M,threads,vgprs", [(0, 256, 72), (0, 512, 72), (64, 256, 96)])
def test_l2_and_l1_scans_keep_their_wavefronts(kernels, M, threads, vgprs, phase):
    k = kernels[f"_ZN3amp6k_scanILi0ELi{M}ELi{phase}ELi1ELi0ELi{threads}EEEvNS_8ScanArgsE"]
    assert k[".private_segment_fixed_size"] == 0
    assert k[".vgpr_count"] <= vgprs


def test_l1_pair_bases_keep_their_wavefronts(kernels):
    k = kernels["_ZN3amp6k_baseILb1EEEvNS_8BaseArgsE"]
    assert k[".private_segment_fixed_size"] == 0
    assert k[".vgpr_count"] <= 72


def test_mixed_class_scans_stay_out_of_scratch(kernels):
    # (M 128 and one-word rows of M 24: a few registers over their waves' share)
    mix = {n: k[".private_segment_fixed_size"] for n, k in kernels.items() if "k_scan_mix" in n}
    assert len(mix) >= 3 * 2 * 16  # phases, granularities, shapes
    few = {"k_scan_mixILi128E": 56, "k_scan_mixILi24E": 20}
    assert not {n: b for n, b in mix.items() if b > max(v * (m in n) for m, v in few.items())}
