"""Interpreter indices are part of the interface (gp_set_variant, gp_stats.variant): new interpreters go to the end."""
from paper_2205_03251_amd import gpeval as g

FIRST = ["f32_k1_s16", "f32_k2_s16", "f32_k4_s16", "f32_k8_s16", "f32_k4_s10", "f32_k8_s10", "f32t_k4_s10", "f32t_k8_s10",
         "f32d_k4_s10", "f32d_k8_s10", "bool_k1_s16", "bool_k2_s16", "bool_k1_s10", "boolw_s10", "boolt_k1_s10",
         "boolt_k2_s10"]


def test_indices_stay():
    names = g.variant_names()
    assert names[:len(FIRST)] == FIRST
    assert len(set(names)) == len(names)
