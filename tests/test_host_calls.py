"""The library's host code without a GPU: what it does when a call of the runtime fails, which launches it makes."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    lib = fake_hip.build(tmp_path_factory.mktemp("fake_hip"))
    return lambda code, **kw: fake_hip.run(lib, code, **kw)


def test_a_failed_call_does_not_fail_the_next_one(host):
    """The runtime hands out a thread's last error until it is asked for; the library reports it once."""
    host("""
        words = np.zeros(50000, np.int32)
        g = pk.Saber(np.r_[0, 500, words.size], words, 1, 100, 0.1, 0.01, 3)
        for call, code, use in (("hipMalloc", -2, lambda: g.set_z(words, 0)), ("hipMemcpy:", -3, lambda: g.counts_nnz()),
                                ("estep_kernel", -2, lambda: g.iterate(1)), ("hipMalloc", -2, lambda: g.token_probs([3]))):
            fake.fake_fail(call.encode(), 1)
            assert code_of(use) == code, call
            g.iterate(1)
            assert g.loglik() == 0.0                # (no kernel has run)
    """)
