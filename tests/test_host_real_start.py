"""The real-weight exact solver started from given potentials returns what it
returns without them (tests/host/real_start_check.cpp, under the sanitizers,
no GPU)."""
import os

from test_host_sanitize import CSRC, HOST, build_and_run, pytestmark  # noqa: F401


def test_started_solves_equal_the_plain_ones(tmp_path):
    out = build_and_run(tmp_path, "real_start_check",
                        [os.path.join(HOST, "real_start_check.cpp"), os.path.join(CSRC, "sk_solver_real.cpp")])
    fields = dict(kv.split("=") for kv in out.split()[1:])
    assert int(fields["solved"]) >= 300 and int(fields["infeasible"]) > 0
