"""What the library's host code asks of the HIP runtime, recorded by a stand-in for it (fake_hip.c: memory is host
memory, kernels do not run): how often a call waits for the device, the limits it sets, and which kernels it falls back
on where there is no memory."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2502_17846_amd", "libgrem.so")

PRELUDE = """
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
fake.fake_text.restype = ctypes.c_char_p
I, L, D = ctypes.c_int32, ctypes.c_int64, ctypes.c_double
keep = []
def mem(n):
    keep.append(ctypes.create_string_buffer(n + 64))
    a = ctypes.addressof(keep[-1])
    return ctypes.c_void_p(a + (-a) % 64)
def reset(limit=2**62):
    fake.fake_reset(ctypes.c_size_t(limit))
def text():
    return [l.split(" ") for l in fake.fake_text().decode().splitlines()]
def stream(n, m, chunks=4):
    return lib.grem_edge_stream_bipartition(ends, ends, L(m), L(n), L(-(-m // chunks)), L(n), big, I(0), big, None, None, None)
def buckets(n, m, k):
    return lib.grem_edge_buckets(ends, ends, L(m), L(n), big, I(k), big, big, big, None)
def partition(n, k, chunk, passes=1, options=None):
    return lib.grem_partition_opt(big, I(32), ends, L(n), I(k), D(1.05), L(chunk), I(passes), None, big, None, None, options, None)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "libamdhip64.so.7")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-w", "-Wl,-soname,libamdhip64.so.7", "-o", out, os.path.join(HERE, "fake_hip.c")],
                   check=True)
    if not os.path.exists(LIB):
        from paper_2502_17846_amd import build
        build.build_library()
    return out


def _run(fake, body, sizes="big, ends = mem(1 << 27), mem(1 << 27)"):
    done = subprocess.run([sys.executable, "-c", PRELUDE + sizes + "\n" + textwrap.dedent(body), fake, LIB], capture_output=True, text=True,
                          timeout=300)
    assert done.returncode == 0, done.stdout + done.stderr


def test_one_read_back_on_the_plain_route(fake):
    _run(fake, """
    for k, chunk in ((8, 10_000), (300, 100_000), (1500, 100_000)):
        for longest, rows in ((10, 0), (50_000, 1), (3_000_000, 7)):
            reset()
            fake.fake_prepass(0, ctypes.c_uint64(longest))
            fake.fake_prepass(16 + 2, ctypes.c_uint64(rows))
            assert partition(100_000, k, chunk) == 0
            t = text()
            assert sum(x[0] == "wait" for x in t) == 1, (k, chunk, longest, t)
            assert any("k_long" in x[1] for x in t) == (longest > 10)
    # more long rows than their list holds: the degree is doubled and the chunks counted again
    reset()
    fake.fake_prepass(0, ctypes.c_uint64(9_000))
    fake.fake_prepass(16, ctypes.c_uint64(50_000))
    fake.fake_prepass(17, ctypes.c_uint64(5))
    assert partition(100_000, 8, 10_000) == 0
    t = text()
    assert sum(x[0] == "wait" for x in t) == 2 and any("k_long_count" in x[1] for x in t)
    """)


def test_a_limit_on_lds_does_not_depend_on_the_call(fake):
    _run(fake, """
    reset()
    for n, m in ((9_000_000, 100_000), (5_000_000, 100_000), (3_000_000, 50_000), (20_000, 50_000), (30_000_000, 9_000_000)):
        assert stream(n, m) == 0
    for n, m, k in ((100_000, 500_000, 128), (100_000, 500_000, 120), (100_000, 500_000, 9), (100_000, 500_000, 30),
                    (20_000_000, 12_000_000, 16), (20_000_000, 12_000_000, 60)):
        assert buckets(n, m, k) == 0
    opt = (ctypes.c_int32 * 8)(3)
    for k in (32, 20, 17, 16, 9, 2):
        for n, chunk in ((300_000, 300_000), (70_000, 20_000)):
            assert partition(n, k, chunk, options=opt) == 0
    for k in (4096, 3000, 1500):
        assert partition(5_000, k, 5_000) == 0
    limits = {}
    for what, kernel, value in text():
        if what == "attribute":
            limits.setdefault(kernel, set()).add(int(value))
    assert len(limits) > 8
    for kernel, values in limits.items():
        assert len(values) == 1, (kernel, values)
    """)


def test_without_the_memory_for_a_faster_form(fake):
    _run(fake, """
    def kernels():
        return " ".join(x[1] for x in text() if x[0] == "launch")
    # n, m: the binned form's pairs are what does not fit
    for limit, binned in ((2**62, True), (140_000_000, False)):
        reset(limit)
        assert stream(5_000_000, 9_000_000, 1) == 0
        t = kernels()
        assert ("k_es_bin" in t) == binned and ("k_es_count" in t) == (not binned)
    for limit, binned in ((2**62, True), (90_000_000, False)):
        reset(limit)
        assert buckets(20_000_000, 12_000_000, 16) == 0
        t = kernels()
        assert ("k_eb_bin" in t) == binned
    for limit, fused in ((2**62, False), (40_000_000, True)):
        reset(limit)
        assert lib.grem_expected_cut(big, I(32), ends, L(12_000_000), big, D(0.1), big, None) == 0
        assert any("k_xc_termsIiLb%d" % fused in x for x in kernels().split())
    for limit, packed in ((2**62, True), (1_000_000, False)):
        reset(limit)
        assert lib.grem_edge_cut_r32(big, ends, L(4_000_000), big, big, None) == 0
        assert ("k_pack_labels" in kernels()) == packed
    # nothing fits: an error, and nothing is left allocated
    reset(1000)
    assert stream(5_000_000, 9_000_000, 1) == -2 and buckets(20_000_000, 12_000_000, 16) == -2
    assert lib.grem_expected_cut(big, I(32), ends, L(12_000_000), big, D(0.1), big, None) == -2
    t = text()
    assert sum(x[0] == "malloc" for x in t) == sum(x[0] == "free" for x in t)
    """, sizes="big, ends = mem(1 << 29), mem(1 << 27)")


def test_edge_chunks_in_as_little_memory_as_the_binned_form_can_do_with(fake):
    # bytes that a binned run takes whose estimates are all doubles, and one less: 17 per node (one with the caller's array), the pairs, 6 to 7 KB per chunk
    _run(fake, """
    def stream(n, m, chunks, counts):
        return lib.grem_edge_stream_bipartition(ends, ends, L(m), L(n), L(-(-m // chunks)), L(n), big, I(0), big, None, big if counts else None, None)
    def bisection(n, m, levels, chunks):
        return lib.grem_recursive_bisection(ends, ends, L(m), L(n), I(levels), L(chunks), D(2.0), big, I(0), big, None)
    for f, a, most in ((stream, (5_000_000, 9_000_000, 4, 1), 26_864_384), (stream, (5_000_000, 9_000_000, 4, 0), 107_080_448),
                       (stream, (4_200_000, 1_000_000, 10, 1), 4_875_776), (stream, (16_000_000, 14_000_000, 1, 1), 140_304_384),
                       (stream, (9_000_000, 3_000_000, 20, 1), 9_260_032), (bisection, (5_000_000, 9_000_000, 3, 10), 404_398_848)):
        reset()
        assert f(*a) == 0 and sum(x[0] == "refused" for x in text()) == 0
        reset(most)
        assert f(*a) == 0, a
        t = text()
        assert sum(x[0] == "refused" for x in t) == 1 and any("k_es_bin" in x[1] for x in t if x[0] == "launch"), (a, t[:4])
        assert not any("k_es_count" in x[1] or "packed" in x[1] for x in t)
    """, sizes="big, ends = mem(1 << 28), mem(1 << 26)")


def test_bucket_tiles_by_edges_and_buckets(fake):
    # tiles of 8,192 edges: 2^25 edges or more, 64 buckets or more, and 6.5e9 edges times buckets
    _run(fake, """
    for m, k, wide in ((2**25 - 1, 32, 0), (2**25, 16, 1), (2**25, 13, 0), (2**25, 2, 0), (45_138_888, 12, 0), (45_138_889, 12, 1),
                       (101_562_499, 8, 0), (101_562_500, 8, 1), (200_000_000, 7, 0), (200_000_000, 1, 0), (2**25, 32, 1)):
        reset()
        assert buckets(50_000, m, k) == 0
        names = [x[1] for x in text() if x[0] == "launch" and "k_eb_scatter" in x[1]]
        assert len(names) == 1 and ("ILi1024E" if wide else "ILi512E") in names[0], (m, k, names)
    """)


def test_estimates_are_packed_by_their_bytes_and_a_tiles_cells(fake):
    # 512 MB of estimates (256 MB from 128 partitions on), and tiles of 2,048 cells: 32 rows of 64, 8 of 256 or of 257
    _run(fake, """
    for n, k, chunk, packed in ((2_200_000, 64, 200_000, 1), (2_200_000, 64, 65_505, 1), (2_200_000, 64, 65_504, 0), (2_200_000, 64, 20_000, 0),
                                (4_200_000, 33, 270_001, 1), (4_200_000, 33, 65_536, 0), (2_000_000, 64, 200_000, 0), (600_000, 128, 20_000, 0),
                                (600_000, 128, 32_753, 1), (300_000, 256, 2_000, 1), (250_000, 256, 100_000, 0), (300_000, 257, 2_000, 1)):
        reset()
        assert partition(n, k, chunk) == 0
        names = {x[1] for x in text() if x[0] == "launch" and "k_score_tile" in x[1]}
        assert len(names) == 1 and ("Lb%dE" % packed) in names.pop(), (n, k, chunk, packed)
    """)


def test_no_exception_where_host_memory_ends(fake):
    # 20 levels: 12.6 MB of counters on the device and as much on the host, of which there is only half
    _run(fake, """
    import resource
    def bisection(levels):
        return lib.grem_recursive_bisection(ends, ends, L(1000), L(1000), I(levels), L(4), D(3.0), big, I(0), big, None)
    assert bisection(2) == 0
    size = int(open("/proc/self/statm").read().split()[0]) * 4096
    resource.setrlimit(resource.RLIMIT_AS, (size + 20_000_000, resource.RLIM_INFINITY))
    reset()
    code = bisection(20)
    resource.setrlimit(resource.RLIMIT_AS, (resource.RLIM_INFINITY, resource.RLIM_INFINITY))
    t = text()
    assert code == -2, code
    assert sum(x[0] == "malloc" for x in t) == sum(x[0] == "free" for x in t)
    """)


def test_the_edge_timing_spans_the_kernels_that_count(fake):
    _run(fake, """
    assert lib.grem_edge_stream_profile_enable(I(1)) == 0
    for n, m, inside in ((20_000, 50_000, {"k_es_count"}), (20_000, 900_000, {"k_es_count"}), (5_000_000, 50_000, {"k_es_bin", "k_es_score_bins"})):
        reset()
        assert stream(n, m, 3) == 0
        t = [x for x in text() if x[0] in ("record", "launch")]
        at = [i for i, x in enumerate(t) if x[0] == "record"]
        assert len(at) == 6
        for a, b in zip(at[::2], at[1::2]):
            got = [x[1] for x in t[a + 1:b]]
            assert len(got) == len(inside) and all(any(k + "E" in g for g in got) for k in inside), got
        ms, steps, edges = D(), L(), L()
        assert lib.grem_edge_stream_profile_read(ctypes.byref(ms), ctypes.byref(steps), ctypes.byref(edges)) == 0
        assert (ms.value, steps.value, edges.value) == (3.0, 3, m)
    """)


def test_the_bench_names_the_edge_kernels_that_run(fake):
    _run(fake, f"""
    sys.path.insert(0, {os.path.dirname(HERE)!r})
    from bench import edge_kernels
    for n, m, chunks in ((20_000, 50_000, 3), ((1 << 22) - 1, 100_000, 2), (1 << 22, 100_000, 2), (1 << 22, 9_000_000, 1), (5_000_000, 16_000_000, 1),
                         (17_000_000, 16_000_000, 1), (17_000_000, 16_000_000, 2), (16_000_000, 16_000_000, 1), (1 << 25, 100_000, 10), (1 << 22, 100_000, 8193)):
        reset()
        c_size = -(-m // chunks)
        chunks = -(-m // c_size)
        assert lib.grem_edge_stream_bipartition(ends, ends, L(m), L(n), L(c_size), L(n), big, I(0), big, None, None, None) == 0
        run = [x[1] for x in text() if x[0] == "launch"]
        for k in ("k_es_count", "k_es_bin", "k_es_ask", "k_es_answer", "k_es_score_bins"):
            assert any(k in x for x in run) == (k in edge_kernels(n, c_size, chunks).split("+")), (n, m, chunks, k)
    """, sizes="big, ends = mem(1 << 28), mem(1 << 26)")
