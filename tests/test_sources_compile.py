"""Every device source passes the compiler's semantic check for gfx950 with the
build's own flags: a form that only one dimension or list length instantiates
must not break the others."""
import os
import shutil
import subprocess

import pytest

from paper_1304_4327_amd import build

pytestmark = pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)),
                                reason="no device compiler")


@pytest.mark.parametrize("src", build.sources(), ids=os.path.basename)
def test_source_compiles(src):
    r = subprocess.run([build.HIPCC, *build.CFLAGS, "-fsyntax-only", src], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
