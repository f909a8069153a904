"""The registers of the library's own kernels, from the metadata of the code
objects that build() embeds in libtri.so: what the comments beside them say
about the wavefronts a SIMD holds (512 vector registers per lane, 800 scalar
registers per SIMD in blocks of 16)."""
import functools
import os
import subprocess

import pytest
import yaml

from tests.conftest import ROOT

LIB = os.path.join(ROOT, "paper_2609_37241_amd", "libtri.so")
LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@functools.lru_cache(maxsize=None)
def kernels(tmp):
    """Demangled kernel name -> its metadata."""
    fat = os.path.join(tmp, "fatbin")
    subprocess.run([os.path.join(LLVM, "llvm-objcopy"), f"--dump-section=.hip_fatbin={fat}", LIB,
                    os.devnull], check=True)
    with open(fat, "rb") as f:
        data = f.read()
    out, at = {}, data.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC) + 8
        for _ in range(int.from_bytes(data[p - 8:p], "little")):
            off, size, n = (int.from_bytes(data[p + 8 * i:p + 8 * i + 8], "little") for i in range(3))
            name = data[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" not in name or not size:
                continue
            co = os.path.join(tmp, "object")
            with open(co, "wb") as f:
                f.write(data[at + off:at + off + size])
            notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", co], check=True,
                                   capture_output=True, text=True).stdout
            meta = yaml.safe_load(notes[notes.index("---"):notes.index("\n...")])
            out.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
        at = data.find(MAGIC, at + 1)
    names = subprocess.run(["c++filt"], input="\n".join(out), check=True, capture_output=True,
                           text=True).stdout.split("\n")
    return {d.removeprefix("void ").split("(")[0]: m for d, m in zip(names, out.values())}


def waves(m):
    """Wavefronts per SIMD that the kernel's registers allow (at most 8)."""
    v, s = -(-m[".vgpr_count"] // 8) * 8, -(-m[".sgpr_count"] // 16) * 16
    return min(8, 512 // v, 800 // s)


@pytest.fixture
def found(tmp_path_factory):
    return kernels(str(tmp_path_factory.getbasetemp()))


CHAINS = [(1, rn, q) for rn in (13, 14, 15) for q in ("false", "true")] + \
         [(dt, rn, "true") for dt in (0, 1) for rn in (11, 12)] + \
         [(0, rn, "true") for rn in (13, 14, 15)]


@pytest.mark.parametrize("inter", ["false", "true"])
@pytest.mark.parametrize("dtype,rn,qkn", CHAINS)
def test_streaming_chains_hold_eight_wavefronts(found, dtype, rn, qkn, inter):
    m = found[f"tri::k_chain<{dtype}, {rn}, 42, {qkn}, {inter}>"]
    assert waves(m) == 8 and m[".vgpr_spill_count"] == 0


@pytest.mark.parametrize("form", ["k_rn_scalar", "k_rn_scalar_res"])
@pytest.mark.parametrize("res", ["false", "true"])
@pytest.mark.parametrize("dtype", [0, 1])
def test_any_alignment_norms_hold_eight_wavefronts(found, form, dtype, res):
    assert waves(found[f"tri::{form}<{dtype}, {res}>"]) == 8


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("inter", ["false", "true"])
def test_qk_norm_rope_holds_six_wavefronts(found, dtype, inter):
    assert waves(found[f"tri::k_rope_vec<{dtype}, true, {inter}>"]) >= 6
