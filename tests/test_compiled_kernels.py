"""What the compiler made of the kernels: properties of the gfx950 assembly that the sources rely on and that no result
shows. Every source is compiled to assembly with the flags the library is built with."""
import os
import re

import pytest

from paper_2603_04135_amd import build as B


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm")
    texts = {}

    def get(src):
        if src not in texts:
            path = str(out / src.replace(".hip", ".s"))
            B._run([B._hipcc(), *B.COMMON_FLAGS, *B.PER_FILE_FLAGS.get(src, []), "--offload-device-only", "-S",
                    os.path.join(B.CSRC, src), "-o", path])
            with open(path) as f:
                texts[src] = f.read()
        return texts[src]

    return get


def _functions(text):
    """Mangled kernel name -> its lines."""
    out = {}
    for m in re.finditer(r"^(_Z\w+):[^\n]*\n(.*?)^\.Lfunc_end", text, flags=re.S | re.M):
        out[m.group(1)] = m.group(2).splitlines()
    return out


@pytest.fixture(scope="module")
def dw_kernel(asm):
    found = [lines for name, lines in _functions(asm("gemm_mfma.hip")).items()
             if "gemm_nt_kernel" in name and "EpiStoreILi0E" in name]
    assert len(found) == 1
    return found[0]


def _waits_for_memory(line):
    return "s_waitcnt" in line and "vmcnt" in line


def test_whole_dw_tile_is_overwritten_without_a_wait(dw_kernel):
    """The 32 stores of a tile that overwrites dW follow each other: no wait for the next tile's slices between them."""
    longest = run = 0
    for line in dw_kernel:
        if "global_store_dwordx4" in line:
            run += 1
            longest = max(longest, run)
        elif _waits_for_memory(line) or "s_cbranch" in line or line.startswith(".LBB") or "global_load" in line:
            run = 0
    assert longest == 32


def test_dw_tile_begins_while_the_stores_of_the_one_before_are_under_way(dw_kernel):
    """From the head of the tile loop to the first product there is no wait for memory: the counted wait in front of
    it leaves the stores of the tile before outstanding."""
    head = next(i for i, line in enumerate(dw_kernel) if "Loop Header: Depth=1" in line and "Inner" not in line)
    first = next(i for i in range(head, len(dw_kernel)) if "v_mfma" in dw_kernel[i])
    assert not [line for line in dw_kernel[head:first] if _waits_for_memory(line)]


@pytest.mark.parametrize("src", ["gemm_f32.hip", "gemm_mfma.hip", "head_kernels.hip", "pack.hip", "select.hip"])
def test_no_kernel_spills_vector_registers(asm, src):
    text = asm(src)
    spills = dict(re.findall(r"\.name: +(_Z\w+)\n.*?\.vgpr_spill_count: (\d+)\n", text, flags=re.S))
    assert spills and {k: n for k, n in spills.items() if n != "0"} == {}


@pytest.mark.parametrize("epilogue,early", [("12EpiLogitsExp", 0), ("13EpiLogitsGrad", 0), ("9EpiLogits", 0),
                                            ("EpiStoreILi1EEELi1ELi1ELi1", 8), ("EpiStoreILi0E", 8)])
def test_where_the_load_addresses_of_a_slice_are_formed(asm, epilogue, early):
    """The steady loop of the vocabulary GEMM starts its products at once and forms each load's address next to the load;
    dH and dW form all eight ahead of the first product. The other way round costs 2 to 3 % of the loop."""
    found = [lines for name, lines in _functions(asm("gemm_mfma.hip")).items()
             if "gemm_nt_kernel" in name and "Li256ELi256" in name and epilogue in name]
    assert len(found) == 1
    ops = [line.split()[0] for line in _steady_loop(found[0]) if re.match(r"\s+[sv]_|\s+ds_|\s+global_", line)]
    assert sum("v_mfma" in op for op in ops) == 64 and ops.count("global_load_lds_dwordx4") == 8
    first = next(i for i, op in enumerate(ops) if "v_mfma" in op)
    formed = sum(op == "v_lshl_add_u64" for op in ops[:first])
    assert formed >= early if early else formed == 0


def _steady_loop(lines):
    """The smallest loop that holds the 64 MFMAs of a slice."""
    labels, best = {}, None
    for i, line in enumerate(lines):
        if m := re.match(r"(\.LBB\d+_\d+):", line):
            labels[m.group(1)] = i
        elif (m := re.search(r"s_cbranch_\w+ (\.LBB\d+_\d+)", line)) and m.group(1) in labels:
            body = lines[labels[m.group(1)]:i + 1]
            if sum("v_mfma" in x for x in body) >= 64 and (best is None or len(body) < len(best)):
                best = body
    return best
