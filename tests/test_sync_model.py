"""The cross-workgroup protocols of the step kernel (grid barrier with epoch
recovery, watchdog, tagged hand-offs and their tag ranges, RMSNorm slices, the
advance of the epoch, the token loop's argmax keys, the reuse of the
per-sequence path's words), modelled with host threads
and std::atomic under ThreadSanitizer, on the library's own protocol arithmetic
(csrc/kl_sync.h).  CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "cpu", "sync_model.cpp")
INC = os.path.join(ROOT, "paper_2410_23668_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("sync") / "sync_model")
    subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=thread", "-pthread", "-DKL_HD=",
                    "-I", INC, "-o", exe, SRC], check=True)
    return exe


def test_protocols_hold_under_thread_sanitizer(model):
    r = subprocess.run([model], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "sync model OK" in r.stdout
    assert "ThreadSanitizer" not in r.stderr


def test_model_catches_a_planted_early_barrier(model):
    # the same check with barrier k waiting for barrier k - 1's target: the
    # model (or ThreadSanitizer) must report it
    planted(model, "--plant-early-barrier")


def test_model_catches_a_chunk_that_waits_for_one_slice(model):
    # a staged chunk that waits for the RMSNorm slice of its first column alone
    planted(model, "--plant-one-slice")


def test_model_catches_an_epoch_advanced_before_every_read(model):
    # workgroup 0 of the step's last phase advances the epoch when it is done
    planted(model, "--plant-early-epoch")


def test_model_catches_keys_cleared_in_their_own_step(model):
    # a token loop whose step clears the argmax keys that it fills itself
    planted(model, "--plant-own-keys")


def test_model_catches_a_reader_that_nothing_waits_for(model):
    # a workgroup without rows in a layer that reads the layer's input
    planted(model, "--plant-idle-reader")


def planted(model, mistake):
    r = subprocess.run([model, mistake], capture_output=True, text=True, timeout=300)
    assert r.returncode != 0
    assert "FAIL" in r.stderr or "ThreadSanitizer" in r.stderr
