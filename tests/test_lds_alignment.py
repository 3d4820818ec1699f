"""Where the dynamic LDS of the kernels starts: behind their static LDS, at a multiple
of the 16 bytes that the widest LDS access takes.  Read from the metadata of the
built library's own code objects."""
import msgpack

from conftest import ensure_hip_lib


def _kernels(path):
    """{name: static LDS bytes} of the kernels in the library's code objects."""
    data = open(path, "rb").read()
    out, at = {}, data.find(b"AMDGPU\0\0")
    while at >= 0:
        # an ELF note: sizes of name and description, type, name, description
        size = int.from_bytes(data[at - 8:at - 4], "little")
        if int.from_bytes(data[at - 4:at], "little") == 32:  # NT_AMDGPU_METADATA
            meta = msgpack.unpackb(data[at + 8:at + 8 + size])
            for k in meta["amdhsa.kernels"]:
                out[k[".name"]] = k[".group_segment_fixed_size"]
        at = data.find(b"AMDGPU\0\0", at + 8)
    return out


def test_dynamic_lds_starts_on_16_bytes():
    kernels = _kernels(ensure_hip_lib().LIBPATH)
    dynamic = {n: s for n, s in kernels.items() if "push_deposit" in n or "fft" in n or "fields_to_k" in n}
    assert len(dynamic) > 40
    assert {n: s for n, s in dynamic.items() if s % 16} == {}
