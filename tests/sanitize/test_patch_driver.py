"""The host code that halves patches, counts working sets and forms row units, under ASan + UBSan and under
ThreadSanitizer (patch_driver.cpp); g++ only: no GPU code is built with a sanitizer."""
import os
import shutil

import pytest

from tests.test_sanitize import HIP_INC, HOST_SRC, build_and_run


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(HIP_INC), reason="g++ or HIP headers missing")
@pytest.mark.parametrize("san", ["address,undefined", "thread"])
def test_patches_and_rows_sanitized(tmp_path, san):
    flags = ["-fsanitize=" + san] + (["-fno-sanitize-recover=all", "-fno-omit-frame-pointer"] if san != "thread"
                                     else [])
    out = build_and_run(tmp_path, "patch_" + san.split(",")[0], [
        "g++", "-std=c++17", "-O1", "-g", *flags, "-D__HIP_PLATFORM_AMD__", "-I" + HIP_INC, "-Iinclude",
        "-Ipaper_2509_00406_amd/csrc", *HOST_SRC, "tests/sanitize/patch_driver.cpp", "-pthread"])
    assert "patch and row checks passed" in out
