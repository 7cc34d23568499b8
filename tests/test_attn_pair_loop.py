"""The committed text of the pair loop (128-query workgroups) is what its generator writes."""
import importlib.util
import os

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_22718_amd", "csrc")


def test_pair_loop_is_what_its_generator_writes():
    spec = importlib.util.spec_from_file_location("gen_attn_loop", os.path.join(CSRC, "gen_attn_loop.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    for kg, name in gen.FILES.items():
        assert gen.render(kg) == open(os.path.join(CSRC, name)).read()
    lines = gen.generate(2)
    # two steps of a tile per wave; the products kept back by the last step stand behind the loop once more
    assert sum(ln.startswith("v_mfma") for ln in lines) == 2 * 32 + gen.DEFER
    assert sum(ln == "s_barrier" for ln in lines) == 2
