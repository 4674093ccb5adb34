"""The compiled code of the walk's checks (gfx950 assembly; no GPU needed)."""
import re

import pytest

from test_kernel_budget import asm, kernel_text  # noqa: F401  (asm: the fixture)


@pytest.mark.parametrize("waves", [7, 8])
def test_a_check_reads_each_header_field_once(asm, waves):  # noqa: F811
    # The table's header is in memory, and a check is a chain of loads: the
    # ridge groups' count (word 5) and stride (word 6) are read once each.
    text = "\n".join(kernel_text(asm, f"ILi{waves}E"))
    for word in (5, 6):
        assert len(re.findall(r"(?:flat|global)_load_dword v\d+, .*\boffset:%d\b" % (4 * word), text)) == 1, word
