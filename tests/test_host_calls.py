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


def test_calls_of_two_threads_on_one_stream_do_not_mix(tmp_path):
    """They share the stream's workspace: between a call's kernel and the sum of
    its slots no other call may be enqueued."""
    run(tmp_path, '''
        shape = (0, 0, 1000000, 8, 8, A, 8, B, 8)
        assert lib.tsg_tsmttsm(*shape, C, 8, S) == 0
        launches()
        def other():
            global t
            t = threading.Thread(target=lambda: lib.tsg_tsmttsm(*shape, C + 4096, 8, S))
            t.start()
            t.join(0.5)   # enough to enqueue its launches, if nothing keeps it
        on("launch", other)
        assert lib.tsg_tsmttsm(*shape, C, 8, S) == 0
        t.join()
        names = [r.name for r in launches()]
        assert [b"fold" in n for n in names] == [False, True, False, True], names
    ''')


def test_launch_sizes_of_long_matrices(tmp_path):
    """A block for every tile as far as a launch goes (fewer than 2^32 work
    items); beyond, fewer blocks, which stride over the tiles."""
    out = run(tmp_path, '''
        name = lambda dt, M, N: lib.tsg_kernel_name(1, dt, 0, M, N)  # beta = 0
        for dt, M, N in [(0, 9, 1), (0, 5, 5), (1, 9, 1), (2, 3, 3), (2, 17, 5), (3, 9, 12)]:
            assert "_once_" in name(dt, M, N) and "_db" not in name(dt, M, N)
            print(name(dt, M, N))
            rows = 16 * int(name(dt, M, N).split("_u")[1].split("_")[0])  # of a wave
            for e in range(20, 35):
                for K in ((1 << e) - 1, 1 << e, (1 << e) + 1):
                    for beta in (0.0, 1.0):
                        assert lib.tsg_tsmm(dt, 0, K, M, N, A, M, C, N, B, N, 1.0, beta, S) == 0, (dt, M, N, K, lib.tsg_last_error())
                        r, = launches()
                        if not r.is_("tsmm_once"):
                            continue
                        assert r.grid * r.block < 1 << 32
                        tiles = -(-K // (rows * (r.block // 64)))
                        assert r.grid == min(tiles, ((1 << 32) - 1) // r.block), (dt, M, N, K, r.grid)
    ''')
    assert "_once_" in out


def test_lds_of_one_kernel_by_calls_of_several_sizes(tmp_path):
    """A kernel whose blocks take more than 64 KB of LDS, by turns more and less
    of it (old rows read or not, narrower and wider matrices)."""
    run(tmp_path, '''
        big = set()
        def sizes(call):
            assert call() == 0, lib.tsg_last_error()
            for r in launches():
                if r.shmem > 64 << 10:
                    big.add((r.name, r.shmem))
        for turn in range(2):
            for dt in range(4):
                for M in range(20, 65, 3):
                    for N in (M, 33, 48, 64):
                        for beta in (1.0, 0.0, 1.0):
                            sizes(lambda: lib.tsg_tsmm(dt, 0, 1 << 24, M, N, A, M, C, N, B, N, 1.0, beta, S))
                        sizes(lambda: lib.tsg_tsmttsm(dt, 0, 1 << 24, M, N, A, M, B, N, C, N, S))
        for kernel in ("tsmm_once", "tsmttsm_stage"):
            names = [n for n, _ in big if kernel.encode() in n]
            assert len(names) > len(set(names)), kernel  # of several sizes
    ''')


def test_row_rule_of_the_one_tile_kernel(tmp_path):
    """Tiles of more than 16 rows from 4096 of them on (with old rows and tiles
    of more than 32 from 6144), of 16 rows at any length but with old rows from
    1024 tiles; where the class's table entry takes such calls."""
    run(tmp_path, '''
        from paper_1905_03136_amd import codegen
        DT = ["r64", "c128", "r32", "c64"]
        reached = 0
        for v in codegen.once_variants():
            c, dt, M, N = v["cfg"], DT.index(v["dt"]), v["maxM"], v["maxN"]
            rows = 16 * c["U"]
            for beta, bit in ((0.0, 2), (1.0, 8)):
                least = (6144 if beta and rows > 32 else 4096) if rows > 16 else 1024 if beta else 0
                took = []
                for K in (rows * least - 1, rows * least, 1 << 24):
                    if K < 1:
                        continue
                    assert lib.tsg_tsmm(dt, 0, K, M, N, A, M, C, N, B, N, 1.0, beta, S) == 0
                    r, = launches()
                    took.append((K, r.is_("tsmm_once")))
                if took[-1][1]:
                    assert c["serves"] & bit
                    assert all(once == (K >= rows * least) for K, once in took), (v, beta, took)
                    reached += 1
                else:
                    assert not any(once for _, once in took)
        assert reached > 400, reached
    ''')


def test_reserved_calls_can_be_captured(tmp_path):
    """After tsg_reserve no call of the shape, any type and arithmetic, has to
    grow the workspace."""
    run(tmp_path, '''
        stream = 100
        for dt in range(6):
            for M, N in [(5, 7), (16, 16), (17, 17), (20, 20), (24, 64), (30, 30), (33, 45), (64, 64)]:
                for K in (3000, 20000, 100000, 1 << 22):
                    stream += 1
                    rec.rec_capturing(0)
                    assert lib.tsg_reserve(dt, K, M, N, stream) == 0
                    rec.rec_capturing(1)
                    for ldb in (N, N + 1, N + 16):
                        assert lib.tsg_tsmttsm(dt, 0, K, M, N, A, M, B, ldb, C, N, stream) == 0, (dt, M, N, K, ldb, lib.tsg_last_error())
    ''')


def test_no_exception_crosses_the_interface(tmp_path):
    """A call whose host allocations fail says so and enqueues nothing; the
    next one works."""
    run(tmp_path, '''
        calls = [lambda: lib.tsg_kernel_name(1, 0, 0, 5, 5), lambda: lib.tsg_workspace_size(0, 0, 1000, 5, 5, 1),
                 lambda: lib.tsg_tsmm(0, 0, 1 << 20, 40, 48, A, 40, C, 48, B, 48, 1.0, 1.0, S),
                 lambda: lib.tsg_tsmttsm(0, 0, 100000, 9, 5, A, 9, B, 5, C, 5, S),
                 lambda: lib.tsg_tsmttsm_noalloc(0, 0, 100000, 9, 5, A, 9, B, 5, C, 5, S),
                 lambda: lib.tsg_reserve(0, 100000, 64, 64, S + 1), lambda: lib.tsg_init(0)]
        rec.rec_out_of_memory(1)
        got = [f() for f in calls]
        rec.rec_out_of_memory(0)
        assert got == ["", 0] + [lib.TSG_E_NOMEM] * 5, got
        assert not launches()
        got = [f() for f in calls]
        assert got[0] and got[1] and got[2:] == [0] * 5, got
    ''')
