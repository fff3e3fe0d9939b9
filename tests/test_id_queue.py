"""CPU test of the spike id queue's protocol (mc_queue.h, the code the
persistent kernel runs): every order of the operations of two claiming
wavefronts and the poller on a queue of two to four slots.  No order may hand
a wavefront another id than the one put in at the position it claimed; the model
sees the fault of a claim that reads its ids only after the exchange."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2111_04398_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("queue") / "id_queue_model")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I" + CSRC, os.path.join(HERE, "id_queue_model.cpp"), "-o", exe],
                   check=True)

    def run(slots, start, adds, per, first, read_first):
        out = subprocess.run([exe, *map(str, (slots, start, adds, per, first, int(read_first)))], check=True,
                             capture_output=True, text=True, timeout=100).stdout.split()
        return [int(x) for x in out]
    return run


# (slots, ids at the start, ids added, smallest claim, first position: 0 or just before the wrap)
@pytest.mark.parametrize("shape", [(2, 2, 1, 1, 0), (2, 1, 2, 1, 0), (4, 4, 2, 2, 0), (1, 1, 1, 1, 0),
                                   (2, 2, 1, 1, 2**32 - 4), (4, 3, 1, 2, 2**32 - 4)])
def test_no_order_loses_an_id(model, shape):
    orders, wrong, most = model(*shape, True)
    assert orders > 1000 and most >= 2 and wrong == 0


def test_the_model_sees_a_read_after_the_claim(model):
    orders, wrong, _ = model(2, 2, 1, 1, 0, False)
    assert orders > 1000 and wrong > 0
