"""Every set of exported calls has its own ABI version, and a library of another
version is refused by its version, not at the first symbol it lacks."""
import re
import os
import subprocess

import pytest

from paper_1410_1629_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
V18 = {"run_photons", "trace_path", "trace_path_noalloc", "peel_off", "backward_density", "backward", "dust_emission",
       "mcrt_tape_bytes", "mcrt_last_error", "mcrt_abi_version"}
CALLS = {18: V18, 19: V18 | {"mcrt_release_workspaces"}, 20: V18 | {"mcrt_release_workspaces", "mcrt_kept_bytes"}}


def test_the_version_names_the_exported_calls():
    assert CALLS[B.ABI_VERSION] == set(B.SYMBOLS)


@pytest.mark.parametrize("version", [18, 19, B.ABI_VERSION + 1])
def test_a_library_of_another_version_is_refused_by_its_version(tmp_path, monkeypatch, version):
    src, lib = tmp_path / "old.c", tmp_path / "libmcrt.so"
    src.write_text("int mcrt_abi_version(void) { return %d; }\n" % version +
                   "".join("int %s(void) { return 0; }\n" % n for n in sorted(V18 - {"mcrt_abi_version"})))
    subprocess.run(["gcc", "-shared", "-fPIC", str(src), "-o", str(lib)], check=True)
    monkeypatch.setattr(B, "LIB_PATH", str(lib))
    monkeypatch.setattr(B, "_lib", None)
    with pytest.raises(RuntimeError, match="ABI version %d, the binding expects %d" % (version, B.ABI_VERSION)):
        B.load()
    assert B._lib is None


def test_the_header_has_the_bindings_version():
    text = open(os.path.join(ROOT, "include", "mcrt.h")).read()
    assert int(re.search(r"#define\s+MCRT_ABI_VERSION\s+(\d+)", text).group(1)) == B.ABI_VERSION
