"""What the kernels' sources have to keep to and no run shows."""
import glob
import os
import re

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
