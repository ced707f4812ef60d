"""What the compiler made of the device code: facts in the metadata of the built library that need no GPU."""
import re

from paper_1611_06256_amd import binding


def scratch_bytes():
    """Kernel -> bytes of scratch memory per thread.  The metadata note of a code object is a msgpack map with its keys in
    order; a kernel's name is followed by this size, one byte for 0 to 127 and a marker above that for anything larger."""
    binding.load_library()
    data = open(binding.lib_path(), "rb").read()
    pairs = re.findall(rb"\.name(?:[\xa0-\xbf]|\xd9.|\xda..)([\x20-\x7e]+)\xbb\.private_segment_fixed_size(.)", data, re.S)
    return {name.decode(): size[0] for name, size in pairs}


def test_no_kernel_needs_scratch_memory():
    # a launch with scratch memory starts about a microsecond later, whether it ever spills or not
    sizes = scratch_bytes()
    assert len(sizes) >= 100 and any("conv12_fused_fwd_kernel" in k for k in sizes)
    assert not {k: v for k, v in sizes.items() if v}
