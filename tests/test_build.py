"""The build's products: what their names stand for, and that nobody can load half of one."""
import os
import stat

import pytest
import torch

from paper_2501_08071_amd import binding
from paper_2501_08071_amd import build as B


def test_the_loaded_binding_is_the_one_of_these_sources_and_this_torch():
    assert binding._fast.__file__ == B.binding_path() and os.path.exists(B.binding_path())


@pytest.mark.parametrize("what", ["torch", "python", "source", "header"])
def test_a_binding_made_from_something_else_has_another_name(what, monkeypatch, tmp_path):
    import sysconfig
    now = B.binding_path()
    if what == "torch":
        monkeypatch.setattr(torch, "__version__", "0.0.1")
    elif what == "python":
        monkeypatch.setattr(sysconfig, "get_config_var", lambda name: ".other-abi.so")
    else:
        # a copy of the sources with one byte more
        root = tmp_path / "root"
        os.makedirs(root / "pkg" / "csrc")
        os.makedirs(root / "include")
        for src, dst in ((os.path.join(B.CSRC, "binding_fast.cpp"), root / "pkg" / "csrc"),
                         *((os.path.join(B.HERE, "..", "include", h), root / "include") for h in ("attn.h", "gemm.h", "rowops.h"))):
            with open(src, "rb") as f, open(dst / os.path.basename(src), "wb") as g:
                g.write(f.read())
        monkeypatch.setattr(B, "HERE", str(root / "pkg"))
        monkeypatch.setattr(B, "CSRC", str(root / "pkg" / "csrc"))
        assert os.path.basename(B.binding_path()) == os.path.basename(now)
        with open(root / "pkg" / "csrc" / "binding_fast.cpp" if what == "source" else root / "include" / "gemm.h", "a") as f:
            f.write("\n")
    assert os.path.basename(B.binding_path()) != os.path.basename(now)


@pytest.mark.parametrize("which", ["binding", "lib"])
@pytest.mark.parametrize("ends", [0, 1])
def test_a_product_takes_its_name_only_when_it_is_complete(which, ends, monkeypatch, tmp_path):
    """A compiler that writes half of its output, looks whether that can be seen under the final name, and ends well or not."""
    out = tmp_path / "product.so"
    cc = tmp_path / "cc"
    cc.write_text(f"""#!/bin/sh
while [ "$1" != "-o" ]; do shift; done
echo half > "$2"
case "$2" in *.so) if [ -e "{out}" ]; then echo seen > "{tmp_path}/seen"; fi; if [ {ends} -ne 0 ]; then exit 1; fi;; esac
echo whole >> "$2"
""")
    cc.chmod(cc.stat().st_mode | stat.S_IXUSR)
    monkeypatch.setenv("CXX", str(cc))
    monkeypatch.setattr(B, "HIPCC", str(cc))
    build = (lambda: B.build_binding(str(out))) if which == "binding" else (lambda: B.build_lib(out=str(out)))
    if ends:
        with pytest.raises(RuntimeError):
            build()
        assert not out.exists()
    else:
        build()
        assert out.read_text() == "half\nwhole\n"
    assert not (tmp_path / "seen").exists() and not list(tmp_path.glob("*.part*"))
