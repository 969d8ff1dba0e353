"""Register use of the GEMM kernels, from the compiler's own report (no GPU): these keep everything in registers.  One spilled register gives a
kernel a scratch segment, which cost every tile of the sparse store kernels 0.15-0.2 us."""
import re

import pytest

UNITS = ["k_fwd", "k_bwd", "k_wgrad", "k_dense_a", "k_dense_b", "k_fp8", "k_fp8_rowwise"]


# translation unit, 2:4 operand, epilogue as the mangled name has it, wave tiles (4 x 4: 256 x 256, 4 x 2: 256 x 128)
@pytest.mark.parametrize("unit,sparse,epilogue,tiles", [
    ("k_fwd", 1, "11EpiRowMajorE", [(4, 4)]),
    ("k_fwd", 1, "17EpiRowMajorMappedE", [(4, 4)]),
    ("k_fwd", 0, "11EpiPrune24TILb0EE", [(4, 4), (4, 2)]),
    ("k_fwd", 0, "11EpiPrune24TILb1EE", [(4, 4), (4, 2)]),              # with the per-feature counts
    ("k_bwd", 0, "10EpiDGatherE", [(4, 4), (4, 2)]),
    ("k_fp8_rowwise", 0, "13EpiPrune24RwTILb0EE", [(4, 4), (4, 2)]),    # with row maxima
    ("k_fp8_rowwise", 0, "13EpiPrune24RwTILb1EE", [(4, 4), (4, 2)]),    # ... and the per-feature counts
    ("k_fp8_rowwise", 0, "12EpiDGatherRwE", [(4, 4), (4, 2)]),
])
def test_kernels_do_not_spill(report, unit, sparse, epilogue, tiles):
    for mi, ni in tiles:
        found = [k for k in report[unit] if f"gemm_kernelILb{sparse}E" in k and epilogue in k and f"Li0ELi{mi}ELi{ni}E" in k]
        assert len(found) == 1, found
        assert report[unit][found[0]] == (0, 0), (found[0], report[unit][found[0]])


# The dense row-wise fp8 epilogues hold a scale a column, a scale a row and the row maxima beside the accumulators: registers that may be spilled.
KNOWN = {("EpiRelu2Rw", 4, 4): 6, ("EpiRelu2Rw", 4, 2): 42, ("EpiDReluRw", 4, 4): 6, ("EpiDReluRw", 4, 2): 8}


@pytest.mark.parametrize("unit", UNITS)
def test_no_other_kernel_spills(report, unit):
    """Every kernel of the unit: also those that read k-major operands, that take two GEMMs or other work into one launch, and every tile."""
    kinds = {"k_fwd": ["gemm_kernel", "gemm_k_major_kernel", "gemm_side_kernel", "gemm_rows_kernel"], "k_bwd": ["gemm_kernel", "gemm_k_major_kernel", "gemm_pair_kernel"],
             "k_wgrad": ["gemm_k_major_kernel", "gemm_duo_kernel"], "k_dense_a": ["gemm_k_major_kernel"], "k_dense_b": ["gemm_k_major_kernel"]}
    for kind in kinds.get(unit, ["gemm_kernel"]):
        assert any(kind in k for k in report[unit]), kind
    bad = {}
    for name, (spilled, scratch) in report[unit].items():
        known = [n for (epilogue, mi, ni), n in KNOWN.items() if "gemm_kernelILb0E" in name and f"{len(epilogue)}{epilogue}E" in name and f"Li0ELi{mi}ELi{ni}E" in name]
        if (spilled or scratch) and not (known and spilled <= known[0]):
            bad[name] = (spilled, scratch)
    assert not bad, bad


@pytest.mark.parametrize("epilogue", ["13EpiPrune24RwTILb0EE", "13EpiPrune24RwTILb1EE", "12EpiDGatherRwE", "10EpiRelu2RwE", "10EpiDReluRwE"])
def test_row_maxima_leave_in_whole_waves(assembly, epilogue):
    """The row maxima of a 256 x 256 tile are 128 words a wave: two instructions of 64 lanes."""
    text = assembly["k_fp8_rowwise"]
    name = re.search(rf"^(_ZN5ffn2411gemm_kernelILb0ENS_{epilogue}E?Lb1ELi0ELi4ELi4E\S*):", text, re.M)[1]
    body = text[text.index(f"\n{name}:"):text.index(f".size\t{name},")]
    assert body.count("global_atomic_umax") == 2


def _body(text, name):
    name = re.search(rf"^(_ZN5ffn24{name}\S*):", text, re.M)[1]
    return text[text.index(f"\n{name}:"):text.index(f".size\t{name},")]


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("keep", [0, 1])
def test_transposed_operands_keep_their_hints(assembly, split, keep):
    """The feature-wise re-compression of the panel form in its two variants: without the streaming hint on the compressed outputs (KEEP), and with it on
    every one (of two features: values, dZ values and metadata each).  Told apart by a value alone, the compiler makes one store of the two."""
    stores = re.findall(r"^\s*global_store_\S+ .*", _body(assembly["k_stream"], f"20featurewise24_kernelILb1ELb{split}ELb{keep}E"), re.M)
    assert sum(" nt" in s for s in stores) == (0 if keep else 6) and len(stores) >= 6


@pytest.fixture(scope="module")
def report(assembly):
    """translation unit -> kernel name -> (spilled registers, bytes of scratch a work item)"""
    kernels = {}
    for unit in UNITS:
        kernels[unit] = {m[1]: (int(m[3]), int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", m[2])[1]))
                         for m in re.finditer(r"\.name:\s+(_Z\S+)\n(.*?)\.vgpr_spill_count:\s+(\d+)", assembly[unit], re.S)}
    return kernels
