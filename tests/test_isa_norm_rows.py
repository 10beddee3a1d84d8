"""Static check of the ISA of the norm's row kernels (CPU only).  Their LDS reads are inline assembly, so nothing but the
hand-written waits keeps an instruction from using a register whose value is still on its way: no vector instruction may touch
the destination of a read that no s_waitcnt lgkmcnt has covered."""
import os
import re
import subprocess

import pytest

import test_isa_waits as T


def _regs(tok):
    tok = tok.rstrip(",")
    m = re.match(r"([va])\[(\d+):(\d+)\]$", tok) or re.match(r"([va])(\d+)()$", tok)
    return frozenset((m.group(1), i) for i in range(int(m.group(2)), int(m.group(3) or m.group(2)) + 1)) if m else frozenset()


def _transfer(state, instructions, hazards, where):
    st = list(state)
    for t in instructions:
        op, toks = t.split()[0], t.split()[1:]
        used = frozenset().union(*(_regs(x) for x in toks)) if op.startswith(("v_", "ds_", "buffer_", "global_")) else frozenset()
        if hazards is not None and any(p & used for p in st):
            hazards.append((where, t))
        if op.startswith("ds_read"):
            st.append(_regs(toks[0]))
        elif op.startswith(("ds_", "s_load", "s_buffer_load")):
            st.append(frozenset())
        elif op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", t)
            if m and int(m.group(1)) < len(st):
                st = st[len(st) - int(m.group(1)):]
        st = st[-40:]
    return tuple(st)


def test_lint_flags_a_copy_before_its_wait(monkeypatch):
    monkeypatch.setattr(T, "_transfer", _transfer)
    code = ["ds_read_b64 v[2:3], v9 offset:0", "v_mov_b32_e32 v5, v3", "s_waitcnt lgkmcnt(0)", "s_endpgm"]
    assert len(T.lint_kernel(code)) == 1
    assert T.lint_kernel([code[0], code[2], code[1], code[3]]) == []


@pytest.mark.skipif(not os.path.exists(T.HIPCC), reason="hipcc not available")
def test_no_register_is_used_before_its_read_has_landed(tmp_path, monkeypatch):
    monkeypatch.setattr(T, "_transfer", _transfer)
    asm = tmp_path / "norm_rows.s"
    cmd = [T.HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-S", "--cuda-device-only", "-o", str(asm), os.path.join(T.ROOT, "paper_2603_22276_amd", "csrc", "norm_rows.hip")]
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert proc.returncode == 0, proc.stdout[-2000:]
    text = asm.read_text()
    kernels = dict(re.findall(r"^(_ZN\S*norm_rows\S*kernel\S*):[^\n]*\n(.*?)^\.Lfunc_end", text, flags=re.S | re.M))
    assert len(kernels) == 12, "six counts of K steps in each of the two 16-bit types"
    assert set(re.findall(r"ScratchSize: (\d+)", text)) == {"0"}
    for name, body in kernels.items():
        assert "v_mfma" in body and not T.lint_kernel(body.split("\n")), name
