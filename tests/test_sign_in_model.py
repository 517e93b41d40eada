"""The workgroups of a launch of k_xcd_rounds agree on which of them share its rounds (csrc/dynlp_signin.h, compiled for the host):
every interleaving of those that choose, sign in, come late or start on another XCD, with the list closed full or before, and slots
that come free only when others have left.  A mistake planted in the model is found."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2604_06596_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("sign_in") / "model")
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__host__=", "-D__device__=", "-I", CSRC, "-o", exe,
                    os.path.join(HERE, "sign_in_model.cpp")], check=True)

    def run(want, own, others, slots, looks, launches, plant=0):
        r = subprocess.run([exe, *map(str, (want, own, others, slots, looks, launches, plant))], capture_output=True, text=True, timeout=120)
        return r.stdout.strip()

    return run


# workgroups wanted, on one XCD, on another, how many of an XCD run at a time, looks at the list before it is closed, launches
@pytest.mark.parametrize("case", [(1, 1, 0, 1, 1, 3), (1, 2, 1, 2, 1, 3), (1, 4, 1, 2, 2, 3), (2, 3, 1, 3, 0, 3), (2, 3, 1, 3, 1, 3),
                                  (2, 3, 1, 3, 2, 3), (2, 3, 1, 1, 2, 3), (2, 3, 2, 2, 1, 2), (3, 3, 0, 3, 0, 3), (3, 4, 0, 3, 2, 3),
                                  (3, 4, 0, 4, 1, 3), (3, 4, 1, 4, 1, 2), (4, 4, 1, 4, 0, 2), (4, 5, 0, 3, 2, 3), (4, 5, 0, 5, 1, 2)])
def test_workgroups_agree_on_who_takes_part(model, case):
    assert model(*case).startswith("ok ")


def test_a_number_that_is_read_after_the_close_leaves_a_wait_without_end(model):
    """Late additions stay in the list: those that read the number from there know of one workgroup more than the one that closed it."""
    assert model(3, 3, 0, 3, 0, 1, 1) == "wrong: a wait that does not end: workgroups disagree on how many they are"


def test_a_launch_number_that_is_left_out_finds_a_closed_list(model):
    assert model(2, 3, 1, 3, 0, 2, 2) == "wrong: no workgroup takes part"
