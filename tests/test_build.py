"""The build without the compiler's optional switches."""
import stat

import pytest

from paper_2408_12677_amd import build


@pytest.mark.parametrize("knows", [True, False])
def test_compiler_without_the_register_form_option(tmp_path, monkeypatch, knows):
    # a stand-in compiler that writes its arguments to the output file, or refuses the option as clang does
    cc = tmp_path / "hipcc"
    refuse = "" if knows else """
case "$*" in *amdgpu-mfma-vgpr-form*)
  echo "clang (LLVM option parsing): Unknown command line argument '-amdgpu-mfma-vgpr-form=1'." >&2; exit 1;;
esac"""
    cc.write_text(f"""#!/bin/sh{refuse}
all="$*"
while [ "$1" != "-o" ]; do shift; done
echo "$all" > "$2"
""")
    cc.chmod(cc.stat().st_mode | stat.S_IXUSR)
    monkeypatch.setenv("HIPCC", str(cc))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libgsr.so"))
    args = open(build.build()).read()
    assert ("amdgpu-mfma-vgpr-form" in args) == knows
    assert "-packed-fp32-ops" in args and "--offload-arch=gfx950" in args
