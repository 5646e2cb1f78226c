"""What the kernels of the built library ask of a launch (their metadata in the code objects): arguments, registers, scratch memory."""
import re
import struct
import subprocess

import pytest

msgpack = pytest.importorskip("msgpack")


def metadata(path):
    """{demangled kernel name: its metadata map} of every gfx950 code object in the library."""
    blob, kernels, at = open(path, "rb").read(), {}, 0
    while (at := blob.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", blob, at + 24)[0]):
            offset, size, length = struct.unpack_from("<QQQ", blob, entry)
            triple = blob[entry + 24:entry + 24 + length]
            entry += 24 + length
            if b"gfx950" in triple and size:
                for k in notes(blob[at + offset:at + offset + size]):
                    kernels[k[".name"]] = k
        at += 24
    names = subprocess.run(["c++filt"], input="\n".join(kernels), capture_output=True, text=True, check=True).stdout.split("\n")
    short = lambda n: re.sub(r"\(anonymous namespace\)::|oases::|^void ", "", n).split("(")[0]
    return {short(re.sub(r"oases::\(anonymous namespace\)::", "", n)): k for n, k in zip(names, kernels.values())}


def notes(elf):
    start, entry, count = struct.unpack_from("<Q", elf, 40)[0], *struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, start + i * entry + 4)
        offset, size = struct.unpack_from("<QQ", elf, start + i * entry + 24)
        at = offset
        while kind == 7 and at < offset + size:   # SHT_NOTE
            n, d, t = struct.unpack_from("<III", elf, at)
            at += 12 + (n + 3) // 4 * 4
            if t == 32:                           # NT_AMDGPU_METADATA
                yield from msgpack.unpackb(elf[at:at + d])["amdhsa.kernels"]
            at += (d + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    from paper_2305_16121_amd import binding
    found = metadata(binding.LIB_PATH)
    assert len(found) > 100
    return found


def test_no_launch_dimensions_among_the_arguments(kernels):
    """A kernel that reads gridDim or blockDim gets 256 more bytes of arguments, which the host fills in at every launch: not the kernels of which a
    pass launches several a layer."""
    some = [n for n in kernels if n.startswith(("gemm_", "bdr_ln_kernel", "cast_bf16_kernel", "attn_", "wave_d", "rope_kernel"))]
    assert len(some) > 80
    for n in some:
        assert not any(a[".value_kind"].startswith("hidden_") for a in kernels[n][".args"]), n


def test_attention_forward_registers(kernels):
    """No scratch memory; and with 64 columns, two query groups and no dropout four workgroups of four waves on a CU: 128 registers of the 512 of a SIMD
    lane, a quarter of the 160 KiB of LDS."""
    forward = {n: k for n, k in kernels.items() if n.startswith("attn_fwd_kernel")}
    assert len(forward) == 16
    for n, k in forward.items():
        assert k[".private_segment_fixed_size"] == 0, n
        if n.startswith("attn_fwd_kernel<64, 2,") and n.endswith("false>"):
            assert k[".vgpr_count"] + k[".agpr_count"] <= 128 and k[".group_segment_fixed_size"] <= 40960, (n, k[".vgpr_count"])


def test_attention_backward_arguments(kernels):
    """A backward that turns nothing back is not given the rotation's table (nor the order of stores that goes with it)."""
    some = {n: k[".kernarg_segment_size"] for n, k in kernels.items() if n.startswith(("attn_bwd_", "attn_dkv", "wave_d"))}
    assert len(some) == 36
    for n, size in some.items():
        assert size == (152 if n.startswith("attn_bwd_rope") else 140 if n.startswith("attn_bwd") else 136), n


def test_gemm_arguments(kernels):
    """A GEMM kernel of one problem is given what it reads: 88 bytes, and 32 more where it adds up its own k slices or leaves row sums behind."""
    some = [n for n in kernels if n.startswith("gemm_") and "group" not in n]
    assert len(some) > 100
    for n in some:
        if n.startswith(("gemm_st", "gemm_pp")):   # <..., epilogue, whole tiles (pp), slices, type of the arguments>
            flags = n[n.index("<") + 1:-1].split(", ")
            more = flags[-2] == "true" or flags[-3] == "8"
            assert flags[-1] == ("GemmCall" if more else "GemmArgs"), n
        assert kernels[n][".kernarg_segment_size"] == (120 if "GemmCall" in n else 88), n


def test_every_kernel_of_the_host_is_in_a_code_object(kernels):
    """The names under which the host asks for kernels are those that the device code has."""
    from paper_2305_16121_amd import binding
    blob = open(binding.LIB_PATH, "rb").read()
    host = blob[:blob.index(b"__CLANG_OFFLOAD_BUNDLE__")]
    asked = {m.decode() for m in re.findall(rb"\0(_ZN5oases12_GLOBAL__N_1\d+\w*_kernelI?[\w$]*)(?=\0)", host)}
    assert len(asked) > 100 and asked <= {k[".name"] for k in kernels.values()}, sorted(asked - {k[".name"] for k in kernels.values()})[:3]
