"""The decode kernel that merges in its last work-group relies on the order of its instructions: partials stored past the XCD's L2,
a wait until they are done, a barrier, and only then the count that lets another work-group read them.  Looked up in the
assembly of this library's own source (no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_06472_amd import build


def test_partials_are_written_through_before_the_count(tmp_path):
    if not shutil.which("hipcc"):
        pytest.skip("needs hipcc")
    asm = str(tmp_path / "decode.s")
    subprocess.run(["hipcc", *build.FLAGS, "-w", "-S", "--cuda-device-only", os.path.join(build.CSRC, "decode_bf16.hip"), "-o", asm],
                   check=True, stderr=subprocess.DEVNULL)
    text = open(asm).read()
    kernels = re.findall(r"^(\S*decode_bf16_kernelILi(?:64|128)ELb1E\S*):.*?^\.Lfunc_end", text, re.M | re.S)
    assert len(kernels) == 2
    for name in kernels:
        body = text[text.index("\n%s:" % name):]
        body = body[:body.index(".Lfunc_end")]
        count = re.findall(r"^\s*(global_atomic_inc.*)$", body, re.M)
        assert len(count) == 1, name
        before, after = body.split(count[0])
        ops = [l.split(";")[0].strip() for l in before.splitlines()]
        ops = [l for l in ops if re.match(r"global_store|s_barrier|s_waitcnt vmcnt\(0\)", l)]
        stores = [i for i, l in enumerate(ops) if l.startswith("global_store") and l.endswith("sc1")]
        assert len(stores) >= 3, name
        assert ops[stores[-1] + 1:][:2] == ["s_waitcnt vmcnt(0)", "s_barrier"], (name, ops[-8:])
        assert not any(l.startswith("global_store") for l in ops[stores[-1] + 1:])
        # and the reader drops what its own caches hold before the first load of a partial
        reader = [l.strip() for l in after.splitlines() if re.match(r"\s*(buffer_inv sc1|global_load)", l)]
        assert reader[0].startswith("buffer_inv sc1"), name


def _kernels(tmp_path):
    """name -> instructions of every decode kernel"""
    if not shutil.which("hipcc"):
        pytest.skip("needs hipcc")
    asm = str(tmp_path / "decode.s")
    subprocess.run(["hipcc", *build.FLAGS, "-w", "-S", "--cuda-device-only", os.path.join(build.CSRC, "decode_bf16.hip"), "-o", asm],
                   check=True, stderr=subprocess.DEVNULL)
    text = open(asm).read()
    out = {}
    for m in re.finditer(r"^(\S*decode_bf16_\w*kernelI\S*):(.*?)^\.Lfunc_end", text, re.M | re.S):
        lines = (l.split(";")[0].strip() for l in m[2].splitlines())
        out[m[1]] = [l for l in lines if l and not l.startswith(".")]
    return out


def test_a_list_that_is_an_argument_is_read_with_the_arguments(tmp_path):
    """Both loads of the list stand before the first wait of the kernels that have it as an argument, and those kernels merge in
    the order that the other ones do."""
    kernels = {n: ops for n, ops in _kernels(tmp_path).items() if "list_kernel" in n}
    assert len(kernels) >= 4
    for name, ops in kernels.items():
        wait = next(i for i, l in enumerate(ops) if l.startswith("s_waitcnt"))
        assert sum(l.startswith("global_load_dwordx3") for l in ops[:wait]) == 2, (name, ops[:wait])
        if not re.search(r"ILi\d+ELb1E", name):
            continue
        (count,) = [i for i, l in enumerate(ops) if l.startswith("global_atomic_inc")]
        near = [l for l in ops[:count] if re.match(r"global_store|s_barrier|s_waitcnt vmcnt\(0\)", l)]
        last = max(i for i, l in enumerate(near) if l.startswith("global_store") and l.endswith("sc1"))
        assert near[last + 1:][:2] == ["s_waitcnt vmcnt(0)", "s_barrier"], (name, near[-8:])
        assert not any(l.startswith("global_store") for l in near[last + 1:])
        reader = [l for l in ops[count:] if re.match(r"buffer_inv sc1|global_load", l)]
        assert reader[0].startswith("buffer_inv sc1"), name


def test_a_form_of_its_own_has_no_other(tmp_path):
    """The kernels of d = 128 hold one instruction for P V each: behind a branch on it every wave, also one without pages, would
    wait for Q.  The one for lists that are arguments, with a merge kernel behind it, holds both: it is the faster form there."""
    kernels = _kernels(tmp_path)
    forms = {}
    for name, ops in kernels.items():
        used = {k for k in ("mfma_f32_4x4x1", "mfma_f32_16x16x4") for l in ops if k in l}
        forms[re.search(r"decode_bf16_\w*kernelI\S*?E(?=Ev)", name)[0]] = len(used)
    assert len(forms) == 14, sorted(forms)
    assert all(n == (2 if "ILi64E" in name or "list_kernelILi128ELb0ELin1E" in name else 1) for name, n in forms.items()), forms
    assert any("list_kernelILi128ELb0ELin1E" in name for name in forms)
