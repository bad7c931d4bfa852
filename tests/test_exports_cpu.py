"""The bindings' lists of entry points are those of the headers."""
import re

import pytest

from paper_2208_05247_amd import denoise, probe, rt3d
from test_library_cpu import HEADER, declared_functions


@pytest.mark.parametrize("header,module", [("rt3d.h", rt3d), ("rt3d_denoise.h", denoise), ("rt3d_probe.h", probe)])
def test_exports_name_every_entry_point(header, module):
    decl = declared_functions(re.sub(r"rt3d\.h$", header, HEADER))
    assert sorted(module.EXPORTS) == decl
