"""The C-ABI library loads and exports every symbol include/sttm.h declares (no GPU needed)."""
import ctypes
import os
import re
import struct

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "sttm.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(sttm_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    from paper_2507_07990_amd import binding
    lib = ctypes.CDLL(binding.LIB_PATH)
    names = _declared()
    assert len(names) >= 12
    for n in names:
        assert hasattr(lib, n), f"{n} declared in sttm.h but not exported"
    assert sorted(binding.EXPORTS) == names


def test_host_side_geometry_helpers():
    from paper_2507_07990_amd import binding as b
    assert b.sttm_nodes_per_frame(16, 16, 1) == 256 + 64 + 16 + 4 + 1
    assert b.sttm_nodes_per_frame(13, 13, 1) == 341          # tables are laid out on the padded grid
    assert b.sttm_nodes_per_frame(14, 14, 4) == 256 + 64 + 16
    assert b.sttm_nodes_per_frame(27, 27, 1) == 1024 + 256 + 64 + 16 + 4 + 1
    assert b.sttm_nodes_per_frame(33, 8, 1) == 0 and b.sttm_nodes_per_frame(8, 8, 3) == 0
    assert b.sttm_node_index(16, 16, 1, 0, 3, 5) == 3 * 16 + 5
    assert b.sttm_node_index(16, 16, 1, 4, 0, 0) == 340
    assert b.sttm_node_index(16, 16, 1, 5, 0, 0) == -1
    assert b.sttm_workspace_bytes(1, 8, 8, 8, 64, b.STTM_F32, 1) > 0
    assert b.sttm_workspace_bytes(1, 8, 8, 8, 60, b.STTM_F32, 1) == 0     # D % 8
    assert b.sttm_workspace_bytes(1, 8, 8, 8, 64, 7, 1) == 0


def _kernel_metadata(path):
    """The metadata of every kernel in a library built by hipcc: its offload bundles, the code objects in them, the
    AMDGPU metadata note (type 32, MessagePack) of each."""
    import msgpack
    blob, magic, kernels = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", []
    for m in re.finditer(magic, blob):
        at = m.start() + len(magic)
        count, = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, at)
            triple = blob[at + 24:at + 24 + n]
            at += 24 + n
            elf = blob[m.start() + off:m.start() + off + size]
            if not triple.endswith(b"gfx950"):
                continue
            phoff, = struct.unpack_from("<Q", elf, 0x20)
            phsize, phnum = struct.unpack_from("<HH", elf, 0x36)
            for i in range(phnum):
                kind, _, start, _, _, length = struct.unpack_from("<IIQQQQ", elf, phoff + i * phsize)
                while kind == 4 and length >= 12:      # PT_NOTE
                    namesz, descsz, note = struct.unpack_from("<III", elf, start)
                    desc = start + 12 + (namesz + 3) // 4 * 4
                    if note == 32:
                        kernels += msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
                    step = desc + (descsz + 3) // 4 * 4 - start
                    start, length = start + step, length - step
    return kernels


def test_no_kernel_uses_scratch_memory():
    """Spilled vector registers or indexed private arrays: a trip to memory in the middle of a kernel, and scratch memory
    that the runtime has to allocate behind the library's back."""
    from paper_2507_07990_amd import binding
    kernels = _kernel_metadata(binding.LIB_PATH)
    assert len(kernels) > 50
    assert {k[".name"]: k[".private_segment_fixed_size"] for k in kernels
            if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]} == {}


def test_kernels_that_use_a_threshold_carry_the_search_they_make_and_no_other():
    """They are built in three kinds, the last template argument: 0 the threshold is known, 1 it is searched among listed
    elements, 2 among all keys. The first has no search's tables in LDS, the second not the third's batch of keys in
    registers (48 is what these kernels took when a search among listed elements was all there was)."""
    from paper_2507_07990_amd import binding
    kernels = _kernel_metadata(binding.LIB_PATH)
    for name, kinds in (("k_temporal_parent", 3), ("k_spatial_decide", 3), ("k_select_tau", 2)):
        kind = {}
        for k in kernels:
            m = re.search(name + r"ILi\d+ELi(\d)EE", k[".name"])
            if m:
                kind.setdefault(int(m[1]), []).append(k)
        assert len(kind) == kinds, name
        assert all(k[".group_segment_fixed_size"] == 0 for k in kind.get(0, [])), name
        assert all(k[".vgpr_count"] <= 48 for k in kind[1]), name
