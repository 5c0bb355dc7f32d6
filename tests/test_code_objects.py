"""The build's checks of its own code objects: they pass on the library that was built and refuse what they are there for."""
import os

import pytest

from paper_2411_08982_amd import check_code
from paper_2411_08982_amd.build import LIB

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="the library is not built")


@pytest.fixture(scope="module")
def texts():
    return list(check_code.code_object_texts(LIB))


def test_token_row_buffers_lie_in_the_first_64_kib(texts):
    assert sum(check_code.check_placement(notes) for notes, _ in texts) >= 9   # three weight formats, three sizes at least


@pytest.mark.parametrize("size,ok", [(65536, True), (66560, True), (65536 + 4096, False), (66560 + 4096, False), (32768, False)])
def test_other_placements_are_refused(size, ok):
    notes = f"""
  - .group_segment_fixed_size: 3072
    .name:           _ZN4lynx11plan_kernelEv
  - .group_segment_fixed_size: {size}
    .max_flat_workgroup_size: 256
    .name:           _ZN4lynx10ffn_kernelILi1ELi2ELi0EEEvNS_9FfnParamsE
"""
    if ok:
        assert check_code.check_placement(notes) == 1
    else:
        with pytest.raises(RuntimeError, match="first 65536"):
            check_code.check_placement(notes)


def test_barriers_wait_for_the_loads_into_lds(texts):
    assert sum(check_code.check_waits(listing) for _, listing in texts) >= 100   # several passes per kernel, two buffers each


@pytest.mark.parametrize("between,wait,ok", [(3, "s_waitcnt vmcnt(3)", True), (3, "s_waitcnt vmcnt(4)", False), (3, "", False),
                                             (3, "s_waitcnt lgkmcnt(0)", False), (0, "s_waitcnt vmcnt(0) lgkmcnt(0)", True),
                                             (5, "s_waitcnt vmcnt(2) lgkmcnt(1)", True)])
def test_a_missing_wait_is_refused(between, wait, ok):
    body = ["buffer_load_dwordx4 v2, s[24:27], 0 offen lds  // 00000000D44C: E05D1000 80060002"]
    body += ["buffer_load_dwordx4 v[4:7], v3, s[28:31], 0 offen nt  // 00000000D474: E05D1000"] * between
    body += [wait + "  // 00000000D494:"] * bool(wait) + ["s_barrier"]
    listing = "0000000000006700 <_ZN4lynx10ffn_kernelILi1ELi2ELi0EEEvNS_9FfnParamsE>:\n" + "\n".join("\t" + l for l in body)
    if ok:
        assert check_code.check_waits(listing) == 1
    else:
        with pytest.raises(RuntimeError, match="nothing waits"):
            check_code.check_waits(listing)
    assert check_code.check_waits(listing.replace("ffn_kernel", "other_kernel")) == 0


def test_operands_of_written_out_products_come_from_loads(texts):
    # two projections, passes of 4, 8, 12 and 16 column tiles, four streams, four k-steps a turn
    assert sum(check_code.check_operands(listing) for _, listing in texts) >= 2 * (4 + 8 + 12 + 16) * 4 * 4


@pytest.mark.parametrize("before,ok", [(["v_mov_b32_e32 v9, v1"], False), (["v_mov_b32_e32 v20, v1", "s_nop 0"], False),
                                       (["v_mov_b32_e32 v9, v1", "s_nop 1"], True), (["v_mov_b32_e32 v12, v1"], True),
                                       (["v_add_u32_e32 v8, v1, v2", "ds_read_b128 v[30:33], v4", "s_waitcnt lgkmcnt(4)"], True),
                                       (["ds_read_b128 v[8:11], v4"], True), (["v_cmp_gt_i32_e32 vcc, v8, v1"], True)])
def test_a_late_write_of_an_operand_is_refused(before, ok):
    body = before + ["v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[20:23], a[0:3]  // 000000008320: D3B580FC"]
    listing = "0000000000006700 <_ZN4lynx15ffn_wide_kernelENS_9FfnParamsE>:\n" + "\n".join("\t" + l for l in body)
    if ok:
        assert check_code.check_operands(listing) == 1
    else:
        with pytest.raises(RuntimeError, match="written"):
            check_code.check_operands(listing)


PRODUCT = "v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[20:23], a[0:3]"


def wide_listing(body, symbol="_ZN4lynx15ffn_wide_kernelENS_9FfnParamsE"):
    """body, four bytes an instruction from 0x6700; "-> n": the target of a branch is the n-th instruction."""
    out = [f"0000000000006700 <{symbol}>:"]
    for i, text in enumerate(body):
        op, _, target = text.partition(" -> ")
        mark = f" <{symbol}+0x{4 * int(target):x}>" if target and int(target) else f" <{symbol}>" if target else ""
        out.append(f"\t{op}{' 0' if target else ''}    // {0x6700 + 4 * i:012X}: BF800000{mark}")
    return "\n".join(out) + "\n"


# A sum of a product is touched too soon (moved, read, stored, loaded over), or written too late; the instructions that exchange two
# registers write both; a write at the end of a loop meets the product at its top, also behind a second branch.
@pytest.mark.parametrize("body,ok", [
    ([PRODUCT, "v_accvgpr_read_b32 v1, a2"], False),
    ([PRODUCT, "v_accvgpr_read_b32 v1, a4"], True),
    ([PRODUCT, "s_nop 15", "s_nop 1", "v_accvgpr_mov_b32 a9, a3"], False),
    ([PRODUCT, "s_nop 15", "s_nop 2", "v_accvgpr_mov_b32 a9, a3"], True),
    ([PRODUCT, "global_store_dwordx4 v[30:31], a[0:3], off"], False),
    ([PRODUCT, "ds_read_b128 a[0:3], v40"], False),
    (["v_accvgpr_write_b32 a3, v1", "s_nop 0", PRODUCT], False),
    (["v_accvgpr_write_b32 a3, v1", "s_nop 1", PRODUCT], True),
    (["v_swap_b32 v1, v9", PRODUCT], False),
    (["v_permlane32_swap_b32_e32 v1, v23", "s_nop 0", PRODUCT], False),
    ([PRODUCT, "v_mov_b32_e32 v9, v1", "s_cbranch_scc1 -> 0", "s_endpgm"], False),
    ([PRODUCT, "v_mov_b32_e32 v9, v1", "s_nop 0", "s_cbranch_scc1 -> 0", "s_endpgm"], True),
    (["s_nop 0", PRODUCT, "s_cbranch_scc0 -> 5", "s_nop 15", "s_nop 15", "s_branch -> 7", "s_endpgm", "v_accvgpr_read_b32 v1, a0"], False),
    ([PRODUCT, "s_branch -> 3", "v_accvgpr_read_b32 v1, a0", "s_endpgm"], True),
])
def test_what_comes_too_close_to_a_product_is_refused(body, ok):
    if ok:
        assert check_code.check_operands(wide_listing(body)) == 1
    else:
        with pytest.raises(RuntimeError, match="states before"):
            check_code.check_operands(wide_listing(body))
    assert check_code.check_operands(wide_listing(body, "_ZN4lynx10ffn_kernelILi1EEEvNS_9FfnParamsE")) == 0
