"""The key under which counters of the step kernel are recorded (CPU only): it
covers every source of the step's launches, and nothing else than their code."""
import os
import re
import shutil

import pytest

import profiling


def included(name, seen):
    seen.add(name)
    with open(os.path.join(profiling.CSRC, name)) as f:
        for inc in re.findall(r'#include "(\w+\.h)"', f.read()):
            if inc not in seen and os.path.exists(os.path.join(profiling.CSRC, inc)):
                included(inc, seen)
    return seen


@pytest.mark.parametrize("unit", ["ddpinn_step.hip", "ddpinn_wide.hip", "ddpinn_api.cpp"])
def test_the_step_s_translation_units_are_covered(unit):
    assert included(unit, set()) <= set(profiling.STEP_SOURCES)


@pytest.mark.parametrize("name", profiling.STEP_SOURCES)
def test_an_edit_of_the_code_changes_the_key_and_one_of_a_comment_does_not(name, tmp_path):
    for f in profiling.STEP_SOURCES:
        shutil.copy(os.path.join(profiling.CSRC, f), tmp_path)
    key = profiling.kernel_source_hash(str(tmp_path))
    assert key == profiling.kernel_source_hash()
    text = (tmp_path / name).read_text()
    (tmp_path / name).write_text("// another comment\n" + text + "\n/* and\n one more */\n")
    assert profiling.kernel_source_hash(str(tmp_path)) == key
    at = text.index("namespace ddp")
    (tmp_path / name).write_text(text[:at] + "constexpr int kOneMore = 1;\n" + text[at:])
    assert profiling.kernel_source_hash(str(tmp_path)) != key


def test_bench_reads_the_key_from_here():
    import bench
    assert bench.traffic_from_profiles("no such workload") is None
    assert not hasattr(bench, "kernel_source_hash")
