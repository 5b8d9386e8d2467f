"""The word exchange of the resident groups, in a host model that runs the kernels' own rules (csrc/wind_group_protocol.h) under schedules a GPU
hardly ever shows: one workgroup held back for as long as any other can move, and random orders."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2505_13765_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("group") / "model")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, os.path.join(HERE, "group_exchange_model.cpp"), "-o", exe], check=True)
    return lambda *args: subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True, timeout=60).stdout.strip()


# column parts, row groups, first iteration without rows in the last row group, iterations between labels
SHAPES = [(32, 1, 0, 7), (3, 1, 0, 50), (1, 1, 0, 13), (31, 1, 0, 1000), (32, 1, 0, 1000), (32, 2, 40, 60), (32, 4, 0, 1000), (10, 4, 25, 9), (32, 2, 40, 1)]


@pytest.mark.parametrize("tag", [1, 0], ids=["bf16", "f32"])
@pytest.mark.parametrize("nparts,rg,empty_from,every", SHAPES)
def test_no_workgroup_misses_or_mistakes_keys(model, nparts, rg, empty_from, every, tag):
    for held in range(32):
        assert model(32, nparts, rg, empty_from, every, held, 0, 1, tag) == "done", held
    for seed in range(8):
        assert model(32, nparts, rg, empty_from, every, -1, seed, 1, tag) == "done", seed


def test_the_model_shows_what_the_rule_is_for(model):
    """Without the rule, workgroups whose keys nobody waits for lose theirs: no column part, no rows left in the row group."""
    assert model(32, 32, 1, 0, 1000, 5, 0, 0, 1) == "done"      # every workgroup has keys that all wait for
    for nparts, rg, empty_from, held in ((3, 1, 0, 20), (32, 2, 40, 31), (32, 4, 0, 24)):
        assert model(32, nparts, rg, empty_from, 1000, held, 0, 0, 1) in ("stuck", "wrong")
        assert model(32, nparts, rg, empty_from, 1000, held, 0, 0, 0) == "stuck"


def test_no_wave_mistakes_the_next_list_of_emitting_slots_for_its_own(tmp_path):
    """Two lists, by the iteration; with one, a wave that is held back reads what the first wave has written for the next iteration."""
    exe = str(tmp_path / "model")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, os.path.join(HERE, "emit_list_model.cpp"), "-o", exe], check=True)

    def run(held, seed, rule):
        return subprocess.run([exe, str(held), str(seed), str(rule)], check=True, capture_output=True, text=True, timeout=60).stdout.strip()

    for held in range(4):
        assert run(held, 0, 1) == "done", held
    for seed in range(8):
        assert run(-1, seed, 1) == "done", seed
    assert run(0, 0, 0) == "done"
    assert [run(held, 0, 0) for held in (1, 2, 3)] == ["wrong"] * 3
