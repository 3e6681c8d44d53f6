"""Where the vocabulary strips of a sweep and the pieces of a contraction begin: the kernels form the quotients
from a factor that the host takes (host code; nothing is launched)."""
from tests import host_program


def test_shares_are_spread_evenly(tmp_path):
    status, out = host_program.run(tmp_path, "shares_main")
    assert status == 0 and out.startswith("ok "), (status, out)
