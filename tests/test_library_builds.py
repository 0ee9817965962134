"""Every source compiles for any number N of martensite variants that the
16-bit constraint masks admit (N is a compile-time constant of a library)."""
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2011_08802_amd import build


@pytest.mark.parametrize("nvar", [1, 4, 5, 8, 13])
def test_sources_accept_any_number_of_variants(nvar):
    """Device pass of the front end (types, templates, static assertions) at
    block sizes 4, 7, 8, 11 and 16: below, beside and above the built ones,
    with padded blocks that are and are not whole groups of 12 entries."""
    def front_end(src):
        return subprocess.run([build.HIPCC, *build.CFLAGS, f"-DMVPF_NVAR={nvar}", "--cuda-device-only", "-fsyntax-only",
                               src], capture_output=True, text=True)
    with ThreadPoolExecutor(4) as ex:
        for src, r in zip(build.sources(), ex.map(front_end, build.sources())):
            assert r.returncode == 0, f"{src}: {r.stderr[-2000:]}"
