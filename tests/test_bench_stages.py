"""The stages that bench.py divides an engine call's kernels into.  CPU only."""
import os
import re

import bench

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2410_09654_amd", "csrc", "engine.hip")

# kernels of an engine call after the records lie in their buckets
AFTER = {"k_merge", "k_merge_small", "k_merge_deferred", "k_norm", "k_scale_filter", "k_plan",
         "k_sel_pass1", "k_sel_narrow", "k_write_out", "k_hist_reduce", "k_select", "k_level1",
         "k_cand_level", "k_finish", "k_count_boundary", "k_scan_buckets", "k_write",
         "k_term_stream", "k_term_bounds"}


def test_every_kernel_of_an_engine_call_has_its_stage():
    text = open(SRC).read()
    run = text[text.index("int Engine::run(Call& c)"):text.index("int dispatch(Engine& e")]
    macros = text[:text.index("int Engine::run(Call& c)")]
    names = set(re.findall(r'\b(?:LAUNCH|EMIT)\(\s*"(k_\w+)"', run + macros))
    assert {"k_emit_sample", "k_scan_wide", "k_emit_append", "k_scan"} <= names
    assert AFTER <= names
    for k in sorted(names):
        assert bench.emission_kernel(k) == (k not in AFTER), k
