"""What the library holds on every GPU for as long as a process lives: the static data of its device
code objects, read from the ELF headers of the built library."""
import struct

from paper_2408_03204_amd import LIB_PATH

EM_AMDGPU, SHF_WRITE, SHF_ALLOC = 224, 1, 2


def device_objects(data: bytes):
    at = data.find(b"\x7fELF", 4)  # after the library's own header
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            yield at
        at = data.find(b"\x7fELF", at + 4)


def writable_bytes(data: bytes, at: int) -> int:
    off, = struct.unpack_from("<Q", data, at + 40)  # e_shoff
    size, count = struct.unpack_from("<HH", data, at + 58)
    total = 0
    for i in range(count):
        _, _, flags, _, _, n = struct.unpack_from("<IIQQQQ", data, at + off + i * size)
        if flags & SHF_WRITE and flags & SHF_ALLOC:
            total += n
    return total


def test_static_device_memory_is_the_scratch_and_little_else():
    """32 MiB of scratch for renders without an allocation, 2 MiB for their delay spectra."""
    data = open(LIB_PATH, "rb").read()
    held = [writable_bytes(data, at) for at in device_objects(data)]
    assert held and 34 << 20 <= sum(held) <= (34 << 20) + (1 << 16), held
