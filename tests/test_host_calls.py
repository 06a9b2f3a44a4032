"""The host side of the library's calls, without a GPU: what it launches and
with which memory (tests/host_calls.py)."""
from .host_calls import run


def test_slots_and_counter_of_a_call_lie_in_one_workspace(tmp_path):
    """A thread that grows the stream's workspace while another one prepares a
    call leaves that call the old workspace or the new one, never parts of both."""
    run(tmp_path, '''
        assert lib.tsg_reserve(0, 1000, 4, 4, S) == 0
        launches()
        def grow():
            t = threading.Thread(target=lambda: lib.tsg_reserve(0, 1 << 22, 64, 64, S))
            t.start()
            t.join()
        on("query", grow)
        assert lib.tsg_tsmttsm(0, 0, 10007, 4, 4, A, 4, B, 4, C, 4, S) == 0
        kernels = [r for r in launches() if r.is_("tsmttsm_")]
        assert len(kernels) == 1
        ws, arrived = kernels[0].args[9], kernels[0].args[11]
        assert arrived == ws + rec.rec_buffer(ws) - 256, (hex(ws), hex(arrived))
    ''')
