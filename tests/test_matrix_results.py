"""The listings of the tiled and the GQA attention: no assembly statement is the first to read what a matrix product wrote.  The compiler spaces its own instructions
behind a product as far as the product's registers need, and nothing before an assembly statement, whose text it does not look at."""
import os
import re
import subprocess

import pytest

from paper_2604_12452_amd import build


def _registers(operand):
    """Names of the vector and accumulation registers of an operand: v7, a[4:7], -v3, |v3|."""
    m = re.fullmatch(r"-?\|?([va])(?:(\d+)|\[(\d+):(\d+)\])\|?", operand)
    if not m:
        return []
    lo, hi = (int(m[2]),) * 2 if m[2] else (int(m[3]), int(m[4]))
    return [f"{m[1]}{i}" for i in range(lo, hi + 1)]


def _blocks(listing):
    """A function's basic blocks in order: [label or None, [(instruction, whether in an assembly statement)]]."""
    blocks, inside = [[None, []]], False
    for line in listing.splitlines():
        if "#ASMSTART" in line or "#ASMEND" in line:
            inside = "#ASMSTART" in line
        label = re.match(r"(\.?\w+):", line)
        text = line.split(";")[0].strip()
        if label:
            blocks.append([label[1], []])
        elif re.match(r"(v|ds|buffer|global|scratch|s)_", text):
            blocks[-1][1].append((text, inside))
            if re.match(r"s_c?branch|s_endpgm", text):
                blocks.append([None, []])
    return blocks


def _step(fresh, text):
    """Registers that a matrix product wrote and nothing has read since, after one more instruction."""
    if text.startswith("s_nop") and int(text.split()[1], 0) >= 15:
        return set(), set()
    if text.startswith("s_"):
        return fresh, set()
    name, *operands = re.split(r"[\s,]+", text)
    named = [_registers(o) for o in operands]
    written = set(named[0]) if name.startswith("v_") else set()
    read = {r for regs in (named[1:] if name.startswith("v_") else named) for r in regs}
    return (fresh | written if name.startswith("v_mfma") else fresh - read - written), read & fresh


def first_reads_in_assembly(listing, own_products=True):
    """Assembly statements of a function that may, on some way through its blocks, be the first to read a register that a matrix product wrote, without a
    wait of their own in between.  own_products=False: of products that the compiler issues (those that are assembly themselves are spaced by hand)."""
    blocks = _blocks(listing)
    at = {b[0]: i for i, b in enumerate(blocks) if b[0]}
    entry, found, todo = [set() for _ in blocks], [], list(range(len(blocks)))
    while todo:
        i = todo.pop(0)
        fresh, last = entry[i], ""
        for text, inside in blocks[i][1]:
            fresh, first = _step(fresh, text)
            if inside and not own_products and text.startswith("v_mfma"):
                fresh, first = fresh - set(_registers(re.split(r"[\s,]+", text)[1])), set()
            if inside and first and text not in found:
                found.append(text)
            last = text
        after = [] if last.startswith(("s_branch", "s_endpgm")) else [i + 1]
        after += [at[last.split()[1]]] if re.match(r"s_c?branch", last) else []
        for j in after:
            if j < len(blocks) and not fresh <= entry[j]:
                entry[j] = entry[j] | fresh
                todo.append(j)
    return found


def test_the_scan_tells_a_first_read_in_assembly():
    product, read = "\tv_mfma_f32_16x16x32_bf16 v[4:7], v[0:3], v[8:11], 0\n", ";;#ASMSTART\n\tv_max_f32 v12, v5, v6\n\t;;#ASMEND\n"
    assert first_reads_in_assembly(product + read) == ["v_max_f32 v12, v5, v6"]
    assert first_reads_in_assembly(product + "\ts_nop 15\n" + read) == []
    assert first_reads_in_assembly(product + "\tv_fma_f32 v5, v5, v20, v21\n\tv_fma_f32 v6, v6, v20, v21\n" + read) == []
    assert first_reads_in_assembly(product + "\tv_fma_f32 v5, v5, v20, v21\n" + read) == ["v_max_f32 v12, v5, v6"]
    around = "\ts_cbranch_scc1 .LBB0_2\n; %bb.1:\n\tv_fma_f32 v5, v5, v20, v21\n\tv_fma_f32 v6, v6, v20, v21\n.LBB0_2:\n"      # (one way of two)
    assert first_reads_in_assembly(product + around + read) == ["v_max_f32 v12, v5, v6"]


def test_no_assembly_statement_reads_a_matrix_product_first(tmp_path):
    out = tmp_path / "attn_tile.s"
    subprocess.run([build.HIPCC, *[f for f in build.FLAGS if f != "-fPIC"], "-S", "--cuda-device-only", os.path.join(build.CSRC, "attn_tile.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    kernels = re.findall(r"^(_ZN?\w*attn_tile_kernel\w+):(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S)
    assert len(kernels) == 16
    for name, listing in kernels:
        assert listing.count("v_mfma_f32") >= 16
        assert first_reads_in_assembly(listing) == [], name


@pytest.mark.parametrize("form", [[], ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]])        # results where the compiler puts them; in vector registers, as it may
def test_no_assembly_statement_of_the_gqa_attention_reads_the_compilers_products_first(tmp_path, form):
    out = tmp_path / "attn_gqa64.s"
    subprocess.run([build.HIPCC, *[f for f in build.FLAGS if f != "-fPIC"], *form, "-S", "--cuda-device-only", os.path.join(build.CSRC, "attn_gqa64.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    kernels = re.findall(r"^(_ZN?\w*attn_gqa64_kernel\w+):(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S)
    assert len(kernels) == 2
    for name, listing in kernels:
        assert first_reads_in_assembly(listing, own_products=False) == [], name
