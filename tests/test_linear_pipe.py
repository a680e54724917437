"""The hand-scheduled 256-row tiles of the linear layers (csrc/linear_pipe.hip): instruction stream (of the loads in the small
tiles' kernels too, csrc/linear.hip) and routes on the CPU, results on the GPU against the float64 oracle."""
import os
import subprocess
import tempfile

import pytest

from paper_2511_19797_amd import build
from tests import dispatch_cases as dc
from tests import test_isa_hazards as isa
from tests.dispatch_rules import ask


def lds_load_violations(asm_text):
    """Buffer loads into LDS take their address from M0: one instruction is due between the scalar write of M0 and the load."""
    ins = list(isa.instructions(asm_text))
    is_load = lambda i: ins[i][0].startswith("buffer_load") and ins[i][1] and ins[i][1][-1].endswith("lds")
    return [i for i in range(1, len(ins)) if is_load(i) and ins[i - 1][0].startswith("s_") and ins[i - 1][1][:1] == ["m0"]]


def test_lds_load_check_sees_a_planted_hazard():
    bad = "s_add_u32 m0, s3, 0\n buffer_load_dwordx4 v1, s[4:7], 0 offen lds"
    assert len(lds_load_violations(bad)) == 1
    assert lds_load_violations(bad.replace("\n", "\n v_add_u32 v1, s2, v3\n")) == []


def generated(name):
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, name + ".s")
        r = subprocess.run(["hipcc", *build.COMMON, *build.PER_FILE.get(name, []), "--cuda-device-only", "-S",
                            os.path.join(isa.CSRC, name), "-o", out], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return open(out).read()


def test_instruction_stream():
    """The rules that no interlock keeps (test_isa_hazards.py), and that nothing spills."""
    text = generated("linear_pipe.hip")
    assert text.count("v_mfma") > 6 * 48
    assert isa.violations(text) == [] and isa.result_violations(text) == [] and lds_load_violations(text) == []
    assert isa.scalar_violations(text) == []
    assert text.count("offen lds") > 100 and "scratch_" not in text


def test_loads_of_the_small_tiles():
    """The 64 and 128 tiles' kernels are the compiler's but for the loads into LDS, which are assembly there too."""
    text = generated("linear.hip")
    assert lds_load_violations(text) == [] and isa.scalar_violations(text) == []
    assert text.count("offen lds") > 100 and "scratch_" not in text


@pytest.mark.parametrize("shape,tiles", dc.LINEAR_PIPE + dc.LINEAR_PITCHED)
def test_routes(shape, tiles):
    (y, gx, gw, _), = ask([("linear", *shape)])
    assert tuple((256, 192, 128, 64)[c] for c in (y, gx, gw)) == tiles


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [c[0] for c in dc.LINEAR_PIPE])
def test_against_the_oracle(shape):
    from tests.test_linear_gpu import run
    run(*shape, seed=1 + shape[0] % 5)
