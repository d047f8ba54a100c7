"""The build takes the compiler as a path, a link or a name on PATH."""
import os

import pytest

from paper_2512_06989_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("how", ["path", "name", "link"])
def test_the_headers_are_found_wherever_hipcc_is(how, monkeypatch, tmp_path):
    hipcc = os.path.realpath(build.HIPCC)
    link = tmp_path / "hipcc"
    link.symlink_to(hipcc)
    monkeypatch.setenv("PATH", os.path.dirname(hipcc) + os.pathsep + os.environ["PATH"])
    monkeypatch.setattr(build, "HIPCC", {"path": hipcc, "name": "hipcc", "link": str(link)}[how])
    assert os.path.exists(os.path.join(build._rocm_include(), "hip", "hip_runtime_api.h"))
