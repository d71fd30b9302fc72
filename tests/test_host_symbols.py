"""Host symbols of the library's sources: a function template that two sources
define under one name with external linkage is one function to the linker,
which keeps either body.  Optimised builds can hide it by inlining one copy, so
the sources are compiled here without optimisation, host side only."""
import collections
import concurrent.futures
import os
import re
import subprocess

import pytest

from paper_2608_01150_amd import build


def _weak(src, tmp):
    obj = os.path.join(tmp, src + ".o")
    flags = [f for f in build.HIP_FLAGS if not f.startswith("-O")]
    subprocess.run([build._hipcc(), "-x", "hip", *flags, "-O0", "--cuda-host-only", "-c", os.path.join(build.CSRC, src),
                    "-o", obj], check=True, capture_output=True)
    out = subprocess.run(["nm", "-C", obj], check=True, capture_output=True, text=True).stdout
    return {m[1] for m in re.finditer(r"^\S+ [WV] (.*)$", out, re.M) if "zl::" in m[1].split("(")[0]}


def test_no_two_sources_define_one_weak_symbol(tmp_path):
    try:
        build._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    with concurrent.futures.ThreadPoolExecutor(8) as ex:
        sets = dict(zip(build.SOURCES, ex.map(lambda s: _weak(s, str(tmp_path)), build.SOURCES)))
    owners = collections.defaultdict(list)
    for src, names in sets.items():
        for n in names:
            owners[n].append(src)
    headers = "".join(open(os.path.join(build.CSRC, h)).read() for h in ("zl_internal.h", "zl_device.h"))
    # inline functions of a header have the one body that every source sees
    base = lambda n: re.split(r"[<(]", n.split("zl::", 1)[1])[0].split("::")[-1]  # noqa: E731
    bad = {n: s for n, s in owners.items() if len(s) > 1 and not re.search(r"\b%s\(" % re.escape(base(n)), headers)}
    assert not bad, bad
