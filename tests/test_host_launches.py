"""What the host layer launches, checked without a GPU: libtlda on a stand-in
for the HIP runtime (tests/host_launches/fake_hip.cpp) that writes launches
down instead of running them."""
import os
import subprocess
import sys

import pytest

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host_launches")
pytest.importorskip("paper_2511_07809_amd.tlda")


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "libamdhip64.so.7")
    script = out + ".map"
    with open(script, "w") as fh:
        fh.write("hip_4.2 { global: *; };\nhip_4.3 { global: hipGraph*; hipStreamBeginCapture;"
                 " hipStreamEndCapture; } hip_4.2;\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7",
                    "-Wl,--version-script," + script, os.path.join(HERE, "fake_hip.cpp"), "-o",
                    out], check=True)
    return out


@pytest.mark.parametrize("check", [
    "fused_grid_does_not_depend_on_the_batch_before",
    "captured_steps_never_regrow_their_partials",
    "no_step_regrows_what_a_graph_writes",
    "rebase_after_a_failed_allocation",
    "classic_step_after_a_failed_allocation",
    "encoder_forward_takes_any_number_of_rows",
    "encoder_tiles_fit_what_they_hold",
    "few_blocks_do_not_form_the_gram_entries",
    "few_columns_take_the_narrow_reduction",
    "short_documents_of_many_topics_keep_the_tall_tiles",
    "small_plans_leave_the_gram_entries_to_the_finish",
    "steps_only_launch",
])
def test_host_launches(stand_in, check):
    r = subprocess.run([sys.executable, os.path.join(HERE, "driver.py"), stand_in, check],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
