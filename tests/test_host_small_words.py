"""What the workgroups of a small frame's ordering say to each other, under every order of their loads and stores (small_words_model.cpp
runs small_words.hpp itself): totals that arrive are those of an ordering with every tile in place."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("model") / "model")
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-I", os.path.join(ROOT, "paper_2511_04283_amd", "csrc"), "-o", out,
                    os.path.join(ROOT, "tests", "small_words_model.cpp")], check=True)

    def run(*args):
        said = subprocess.run([out, *map(str, args)], check=True, capture_output=True, text=True).stdout.split()
        return dict(zip(("schedules", "wrong", "whole", "given_up", "placed_late"), map(int, said)))
    return run


@pytest.mark.parametrize("tile, totals", [(1, 1), (1, 2), (2, 1), (2, 2), (1, 3)])
def test_totals_mean_that_every_tile_is_in_place(model, tile, totals):
    got = model(tile, totals, 0)
    assert got["wrong"] == 0
    # (the orders that it is about were among them: calls that end whole, that are given up, and a tile that looks once more)
    assert min(got["whole"], got["given_up"], got["placed_late"]) > 0, got


def test_a_word_taken_back_may_have_been_seen(model):
    """The model finds the orders in which a tile that takes its word back is missing from totals that count it."""
    assert model(1, 2, 1)["wrong"] > 0
