"""What the compiler made of the kernels: properties that the source asks for, that results do not show and that an
optimiser may undo without a sign.  Reads the gfx950 code of the library as it was built (no GPU)."""
import os
import re
import struct
import subprocess

import pytest

from paper_1511_02490_amd import build, libstencil  # noqa: F401  (loads, and so builds, the library)

LLVM = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")))), "llvm", "bin")


class Kernels:
    """The library's kernels: demangled name -> (code object, symbol, vector registers)."""

    def __init__(self, path, folder):
        data = open(path, "rb").read()
        self.found = {}
        magic = b"__CLANG_OFFLOAD_BUNDLE__"
        at = data.find(magic)
        while at >= 0:
            pos = at + len(magic) + 8
            for _ in range(struct.unpack_from("<Q", data, at + len(magic))[0]):
                off, size, n = struct.unpack_from("<QQQ", data, pos)
                if b"gfx950" in data[pos + 24:pos + 24 + n]:
                    self._add(os.path.join(folder, "%d.elf" % at), data[at + off:at + off + size])
                pos += 24 + n
            at = data.find(magic, at + 1)

    def _add(self, path, code):
        with open(path, "wb") as fh:
            fh.write(code)
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", path], capture_output=True, text=True, check=True).stdout
        kernels = re.findall(r"\.name:\s+(_Z\S+)\n(?:.*\n)*?.*\.vgpr_count:\s+(\d+)", notes)
        names = subprocess.run(["c++filt"], input="\n".join(k for k, _ in kernels), capture_output=True, text=True, check=True).stdout
        for (symbol, vgprs), name in zip(kernels, names.splitlines()):
            self.found[name.split("(")[0].replace("void ", "").replace("sk::", "")] = (path, symbol, int(vgprs))

    def matching(self, pattern):
        return {name: k for name, k in self.found.items() if re.search(pattern, name)}

    def instructions(self, pattern):
        """name -> list of instructions (mnemonic and operands) of every kernel whose name matches."""
        by_file, out = {}, {}
        for name, (path, symbol, _) in self.matching(pattern).items():
            by_file.setdefault(path, {})[symbol] = name
        for path, symbols in by_file.items():
            text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn",
                                   "--disassemble-symbols=" + ",".join(symbols), path], capture_output=True, text=True, check=True).stdout
            for block in re.split(r"\n(?=[0-9a-f]+ <)", text)[1:]:
                lines = block.splitlines()
                out[symbols[re.search(r"<(.+)>:", lines[0]).group(1)]] = [re.sub(r"\s*//.*", "", l).strip() for l in lines[1:]]
        return out


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    return Kernels(build.LIB_PATH, str(tmp_path_factory.mktemp("code")))


def vector_stores(instructions):
    """(plain, non-temporal) 16-byte stores to global memory."""
    stores = [i for i in instructions if i.startswith("global_store_dwordx4")]
    nt = sum(1 for i in stores if i.endswith(" nt"))
    return len(stores) - nt, nt


def test_marching_kernels_store_as_they_were_compiled_to(kernels):
    """The marches over rows of whole vectors exist once for plain and once for non-temporal stores, those of four to eight
    applications for written-through ones too; and of the marches of one application those that the rule can choose:
    sin/cos, 5x5, two to nine columns of up to five rows and seven to nine of up to eleven."""
    code = kernels.instructions(r"^(stream_kernel<.*, true, (true|false), 256>|march_kernel<.*>|march_masked_kernel<.*>)$")
    assert len(code) == 2 * (2 * 2 * 8 + 3 * 2 + 3 * (8 + 3))
    for name, instructions in code.items():
        plain, nt = vector_stores(instructions)
        assert (plain, nt > 0) == (0, True) if name.endswith(", true, 256>") else (plain > 0, nt) == (True, 0), (name, plain, nt)
    through = kernels.instructions(r"^stream_through_kernel<")
    assert len(through) == 2 * 2 * 5
    for name, instructions in through.items():
        stores = [i for i in instructions if re.match("(global|buffer)_store", i)]
        assert stores and all(i.startswith("buffer_store_dwordx4") and i.endswith(" offen sc1") for i in stores), name


def test_kernels_that_choose_at_run_time_keep_both_kinds_of_store(kernels):
    """A plain and a non-temporal store differ in nothing else, and a compiler that merges them leaves plain ones."""
    code = kernels.instructions(r"^(tile_kernel<OpWeightedSum, |tile_kernel<OpSinCos, |direct_kernel<OpHeat, |temporal_kernel<OpHeat, |"
                                r"life_temporal_kernel<|life_direct_kernel<|life_stream_kernel<.*, false>)")
    checked = 0
    for name, instructions in code.items():
        if re.match(r"tile_kernel<.*, \d+, 1, \d+>$", name):
            continue                               # one cell per work-item and row: no vectors
        plain, nt = vector_stores(instructions)
        assert plain > 0 and nt > 0, (name, plain, nt)
        checked += 1
    assert checked > 60


def test_written_through_tiles_write_vectors_through(kernels):
    """Every tile and direct kernel that is there once more to write its output through does so with all its 16-byte stores."""
    code = kernels.instructions(r"^(tile|direct)_kernel<WrittenThrough<")
    assert len(code) >= 120
    plain = kernels.matching(r"^(tile|direct)_kernel<(?!WrittenThrough)")
    for name, instructions in code.items():
        vectors = [i for i in instructions if re.match("(global|flat|buffer)_store_dwordx4", i)]
        assert vectors and all(i.startswith("global_store_dwordx4") and i.endswith(" sc1") for i in vectors), name
        assert re.sub(r"WrittenThrough<(\w+) ?>", r"\1", name) in plain, name


def test_life_streams_write_whole_lines_through(kernels):
    """Bytes that are written through are handed to the lane whose neighbours store the bytes beside them."""
    code = kernels.instructions(r"^life_stream_kernel<.*, false>$")
    assert len(code) == 3 * 4 * 2
    for name, instructions in code.items():
        moves = sum(i.startswith("ds_bpermute_b32") for i in instructions)
        through = sum(i.startswith("global_store_dwordx4") and " sc1" in i for i in instructions)
        assert through == moves > 0, (name, through, moves)


def test_heat_marches_keep_their_wavefronts(kernels):
    """A SIMD's 512 vector registers hold this many wavefronts of a heat march of so many steps per launch."""
    for border, depth, waves in [(1, 5, 5), (1, 7, 4), (2, 5, 5), (2, 7, 4), (1, 8, 3), (2, 8, 4)]:
        found = kernels.matching(r"^(stream_kernel<OpHeat, %d, %d, true, |stream_through_kernel<OpHeat, %d, %d, )" % (border, depth, border, depth))
        assert len(found) == 3                   # plain, non-temporal and written-through stores
        for name, (_, _, vgprs) in found.items():
            assert 512 // ((vgprs + 7) // 8 * 8) >= waves, (name, vgprs)


def test_window_rows_are_read_in_vectors(kernels):
    """Tiles of bytes and of two planes: what a work-item reads of a window row are 16-byte vectors (12 of their bytes
    where the last cell is not needed) and, of bytes, the cells beside them."""
    for pattern, pieces in [(r"^tile_kernel<OpLife, ., .*, 16, \d+>$", {"ds_read_b128", "ds_read_u8"}),
                            (r"^tile_kernel<OpSinCos, ., HaloC<.*, 4, \d+>$", {"ds_read_b128", "ds_read_b96"})]:
        code = kernels.instructions(pattern)
        assert len(code) == 12
        for name, instructions in code.items():
            assert {i.split()[0] for i in instructions if i.startswith("ds_read")} <= pieces, name


def test_folds_of_few_taps_keep_their_wavefronts(kernels):
    """The tap-by-tap tiles with four rows of cells are kernels of their own: 8 wavefronts per SIMD (int32: 6)."""
    for pattern, limit in [("OpWeightedSum, ., HaloTaps, 4, 4,", 64), ("OpWeightedSumF64, ., HaloTaps, 4, 2,", 64),
                           ("OpWeightedSumU8, ., HaloTaps, 4, 4,", 64), ("OpWeightedSumI32, ., HaloTaps, 4, 4,", 80)]:
        found = kernels.matching("^tile_kernel<" + pattern)
        assert len(found) == 3
        for name, (_, _, vgprs) in found.items():
            assert vgprs <= limit, (name, vgprs)


def memory_loads(instructions):
    """Loads from global memory into vector registers."""
    return sum(1 for i in instructions if i.startswith("global_load") and not i.startswith("global_load_lds"))


def test_weights_of_run_time_regions_are_scalar_loads(kernels):
    """The tap-by-tap tiles load into vector registers what the tiles that fold in blocks do: the cells they stage."""
    taps, blocks = kernels.instructions("^tile_kernel<.*HaloTaps"), kernels.instructions("^tile_kernel<.*HaloBlocks")
    assert len(taps) >= 45
    for name, instructions in taps.items():
        assert memory_loads(instructions) == memory_loads(blocks[name.replace("HaloTaps", "HaloBlocks")]), name


def test_tiles_of_single_cells_stage_at_ordinary_priority(kernels):
    """... and, with nothing before the fold that could write to memory, read the weights by scalar loads: the one vector
    load is the staging's."""
    code = kernels.instructions(r"^tile_kernel<.*, 1, \d+>$")
    assert len(code) >= 60
    for name, instructions in code.items():
        assert not any(i.startswith("s_setprio") for i in instructions), name
        assert memory_loads(instructions) == 1, name
