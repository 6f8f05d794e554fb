"""The kernels' resource figures, as the built library's code objects state them."""
import msgpack
import pytest

from paper_2512_05831_amd import build


def kernels():
    """Every kernel's metadata: the AMDGPU notes (type 32) of the code objects in the library."""
    with open(build.LIB, "rb") as f:
        blob = f.read()
    found, at = [], blob.find(b"AMDGPU\0\0")
    while at >= 0:
        namesz, descsz, kind = (int.from_bytes(blob[at - 12 + 4 * i:at - 8 + 4 * i], "little") for i in range(3))
        if namesz == 7 and kind == 32:
            found += msgpack.unpackb(blob[at + 8:at + 8 + descsz], strict_map_key=False)["amdhsa.kernels"]
        at = blob.find(b"AMDGPU\0\0", at + 1)
    return found


@pytest.mark.parametrize("name", ["eb_gather_wave", "eb_gather_plain"])
def test_ragged_rows_spill_no_registers(name):
    """The kernels that rows of any size take keep their sums in registers: no scratch memory."""
    ks = [k for k in kernels() if name in k[".name"]]
    assert len(ks) >= 12
    spilled = {k[".name"]: k[".private_segment_fixed_size"] for k in ks
               if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert not spilled
