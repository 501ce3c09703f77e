"""The host runtime without a GPU: what it does when the system refuses something, and which launches it chooses."""
import pytest

from tests import host_stub


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_stub.build(str(tmp_path_factory.mktemp("stub") / "libpb_stub.so"))


def test_read_back_without_the_threads_it_asks_for(lib):
    """4.7 million parameters, ten chunks through the ring of eight: unpacked by as many threads as there are."""
    host_stub.run(lib, """
from oracle import pb_oracle as O
net = mlp(2048, 2300, 12)
e, want = engine(net), O.PBOracle(net).read_weights().astype(np.float32)
for refused in (0, 1, 2, 100):
    put('threads_refused', refused)
    assert np.array_equal(e.read_weights(), want), refused
e.close()
""")
