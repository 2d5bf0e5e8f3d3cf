"""What the kernels' sources have to keep to and no run shows."""
import glob
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_04283_amd", "csrc")


def text(name):
    return open(os.path.join(CSRC, name)).read()


def test_parameters_that_a_training_iteration_writes_are_not_restrict():
    """k_preprocess_bwd updates in place (train.p) the arrays it also reads as means, scales, quats, opac and sh."""
    signature = re.search(r"void k_preprocess_bwd\((.*?)\)\s*\n\{", text("preprocess.hip"), re.S).group(1)
    signature = re.sub(r"/\*.*?\*/", "", signature, flags=re.S)
    for name in ("means", "scales", "quats", "opac", "sh"):
        declared = [a.strip() for a in signature.split(",") if a.split()[-1] == name]
        assert declared == [f"const float* {name}"], declared


def test_inline_assembly_gives_back_the_lanes_it_found():
    """Assembly that narrows the lane mask saves the one it found and restores that, not a constant: it may stand where some
    lanes are inactive."""
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        for block in re.findall(r"\basm\b[^;]*;", open(path).read()):
            code = "".join(re.findall(r'"([^"]*)"', block))
            if not re.search(r"\bexec\b|saveexec", code):
                continue
            seen += 1
            steps = [line.strip() for line in code.replace("\\t", "").split("\\n")]
            saved = re.match(r"s_and_saveexec_b64 (%\[\w+\]), ", steps[0])
            assert saved, (path, steps[0])
            restored = steps[-1].split("=")[0]
            assert restored.startswith(f"s_mov_b64 exec, {saved.group(1)}"), (path, restored)
            assert not any("exec" in line for line in steps[1:-1]), path
    assert seen == 1


def test_multiply_add_rate_is_measured_on_vector_registers():
    """fs_measure_peaks times chains of multiply-adds as the fastest that the kernels could issue.  One that reads a scalar register
    takes nearly twice as long on this chip as one of vector registers only, and a kernel's arguments arrive in scalar ones."""
    from paper_2511_04283_amd import build
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    asm = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "-w", "-I", os.path.join(build.ROOT, "include"), "-I", CSRC,
                          "--cuda-device-only", "-S", "-o", "-", os.path.join(CSRC, "optimizer.hip")], check=True, capture_output=True,
                         text=True).stdout
    kernel = re.search(r"^\w*k_fma_chain\w*:(.*?)s_endpgm", asm, re.S | re.M).group(1)
    chains = re.findall(r"^\s+(v_fma\w*)\s+(.*)$", kernel, re.M)
    for name, operands in chains:
        assert all(re.fullmatch(r"v\d+", o.strip()) for o in operands.split(";")[0].split(",")), (name, operands)
    # (and no other vector instruction between them)
    loop = re.search(r"^(\.\w+):[^\n]*\n((?:(?!^\.\w+:).)*?)s_cbranch_\w+ \1", kernel, re.S | re.M).group(2)
    work = [line.split()[0] for line in loop.splitlines() if line.strip() and not line.strip().startswith(";")]
    assert sum(w.startswith("v_fma") for w in work) >= 64 and sum(w.startswith("v_") and not w.startswith("v_fma") for w in work) == 0, work
