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
    assert sum(check_code.check_placement(notes) for notes in texts) >= 9   # three weight formats, three sizes at least


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
