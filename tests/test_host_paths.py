"""What the library's host code launches, allocates and gives back, seen by a
program that stands in for the HIP runtime (host/fake_hip.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2005_12489_amd")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    lib = os.path.join(PKG, "libhv.so")
    if not os.path.exists(lib):
        import __graft_entry__
        __graft_entry__.build()
    out = str(tmp_path_factory.mktemp("host") / "fake_hip")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), os.path.join(HERE, "host", "fake_hip.cpp"), lib,
                    "-Wl,-rpath," + PKG, "-L/opt/rocm/lib", "-Wl,--allow-shlib-undefined", "-lpthread", "-o", out],
                   check=True)
    return out


def talk(exe, *lines):
    """The answers to commands: a list of words each."""
    p = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=100)
    assert p.returncode == 0, p.stderr
    answers = [a.split() for a in p.stdout.splitlines()]
    assert len(answers) == len(lines), p.stderr
    return answers


def kernels(answer):
    """[(name, workgroups, threads)] of a call's launches, the call having succeeded."""
    assert answer[0] == "0"
    return [(f[0], int(f[1]), int(f[2])) for f in (w.rsplit(":", 3) for w in answer[1:])]


def names(answer):
    return [k[0].split("<")[0] for k in kernels(answer)]


@pytest.mark.parametrize("call", ["batch", "aa"])
def test_small_explicit_batches(exe, call):
    """In another shape than the default's, a few requests of small indexes take two
    launches: the object kernel's costs more than its strips save."""
    two, three = ["k_tile_frontier", "k_query_region"], ["k_tile_frontier", "k_query_objects", "k_query_region"]
    for n, requests, want in ((65_535, 16, two), (65_535, 17, three), (65_536, 1, three)):
        _, a = talk(exe, f"build p 0 {n}", f"{call} p 4 {requests} 32 1 2 128 0")
        assert names(a) == want, (n, requests)


@pytest.mark.parametrize("call,index,shape", [("batch", "build p 0 100000", "32 4 2 512"), ("aa", "build p 1 100000", "32 4 2 512"),
                                              ("fill", "polygons p 30000", "32 2 2 128"), ("fill", "polygons p 30000", "64 4 2 256")])
def test_asked_for_workgroups(exe, call, index, shape):
    """A persistent kernel of grid_wgs workgroups has that many, in small calls too."""
    for n in (1, 40, 64, 65):
        _, a, b = talk(exe, index, f"{call} p 4 {n} {shape} 7", f"{call} p 4 {n} {shape} 0")
        assert kernels(a)[-1][1] == 7, f"{n} requests: {kernels(a)}"
        assert kernels(b)[-1][1] >= 4 * n, f"{n} requests: {kernels(b)}"


@pytest.mark.parametrize("call", ["batch p 4 3000", "batch p 4 50", "aa p 4 2000", "aa p 0 100 32 1 2 128 0", "batcher b 20000"])
def test_kept_memory_makes_way(exe, call):
    """Memory kept for the next build is given back before an allocation of a call
    that renders, or of a batcher, fails."""
    lines = ["build p 0 2000000", "build q 1 6000000", "free q", "memory"]
    held = int(talk(exe, *lines)[-1][1])
    answers = talk(exe, *lines, f"limit {held + 1000}", call, "limit 1", call)
    assert answers[5][0] == "0"
    assert answers[7][0] != "0"


def test_trim(exe):
    """hv_trim gives back what hv_free kept, and nothing of what is in use."""
    a = talk(exe, "build p 0 200000", "trim", "memory", "build q 1 3000000", "polygons r 300000", "free q", "free r",
             "memory", "trim", "memory", "batch p 4 100", "free p", "trim", "memory")
    assert int(a[7][1]) > int(a[2][1])
    assert a[9][1] == a[2][1]
    assert a[10][0] == "0" and a[13][1] == "0"


def test_pool_threads(exe):
    """Threads that build and free at once: every block is given out once, and all
    of them, at most 1 GiB kept, can be given back."""
    a = talk(exe, "threads 8", "memory", "trim", "memory")
    assert a[0] == ["0"]
    assert 0 < int(a[1][1]) <= 1 << 30 and a[3][1] == "0"


@pytest.mark.parametrize("first,then", [("build a 1 4000000", "build b 1 2500000"), ("polygons a 600000", "polygons b 390000")])
def test_device_bytes(exe, first, then):
    """hv_info's device_bytes are what indexes hold, also in reused blocks."""
    a = talk(exe, "build p 0 300000", first, "trim", "memory", "free a", then, "trim", "memory")
    assert int(a[0][1]) + int(a[1][1]) == int(a[3][1])
    assert int(a[0][1]) + int(a[5][1]) == int(a[7][1])


@pytest.mark.parametrize("build", ["build p 0 2000000", "build p 1 2000000", "polygons p 600000"])
def test_without_memory_for_cells(exe, build):
    """The occupancy cells are an aid: an index is built without them where their
    block does not fit, and holds what it would otherwise less that block."""
    with_cells, memory = talk(exe, build, "memory")
    most, whole = int(memory[2]), int(with_cells[1])
    held = {whole}
    for limit in range(most - 1, whole // 2, -max(1, most // 97)):
        a = talk(exe, f"limit {limit}", build, "trim", "memory")
        if a[1][0] != "0":
            assert a[3][1] == "0"  # and nothing is left of a failed build
            break
        held.add(int(a[1][1]))
        assert a[1][1] == a[3][1]
    assert len(held) == 2, held


def test_autotune_candidates(exe):
    """Every shape is timed once (a first run and three on the whole sample), but for
    those that differ in the cull depth, which the launch does not show; one wave with
    a workgroup to a region and persistent; and of equals the default is taken."""
    _, a = talk(exe, "build p 0 3000000", "tune p 6 4096")
    assert a[:2] == ["0", "32:1:2:96:0"]
    count = {}
    for w in a[2:]:
        if "region" in w or "both" in w:
            count[w] = count.get(w, 0) + 1
    whole = {w: c for w, c in count.items() if int(w.rsplit(":", 3)[1]) > 128 * 64}  # (not the parts of the sample)
    assert sorted(set(whole.values())) == [4, 8, 12], whole
    assert list(whole.values()).count(12) == 1 and list(whole.values()).count(8) == 1, whole
    one_wave = [w.rsplit(":", 3) for w in whole if w.rsplit(":", 3)[2] == "64" and "<32,2," in w]
    lds = sorted({f[3] for f in one_wave})
    assert len(lds) == 3 and len(one_wave) == 6, one_wave  # queues of 64, 96, 128, two grids each


@pytest.mark.parametrize("n,dense,waves", [(1, 1, 4), (1023, 1023, 4), (1024, 255, 4), (1024, 256, 2), (4095, 4095, 2),
                                           (4096, 1023, 2), (4096, 1024, 1), (9000, 0, 4), (9000, 255, 4), (9000, 256, 2),
                                           (9000, 9000, 1)])
def test_waves_by_size_and_density(exe, n, dense, waves):
    """The default's waves per region follow the batch's size and how many of its
    requests lie in dense data, in a batcher's graphs as in a call; a batcher too
    small for a class of sizes takes the next."""
    # 16,384 objects a tile and more count as dense: 300,000 at zoom 2
    _, b, small, a, c, d = talk(exe, "build p 0 300000", "batcher b 10000", "batcher s 3000",
                                f"run p b 2 {n} {dense}", f"run p s 2 {min(n, 3000)} {min(dense, 3000)}",
                                f"batch p {2 if dense else 22} {n}")
    assert b == ["0"] and small == ["0"]
    assert kernels(a)[-1][2] == 64 * waves, kernels(a)
    assert kernels(c)[-1][2] == 64 * max(waves, 2), kernels(c)
    if dense in (0, n) and n > 64:
        assert kernels(d)[-1][2] == 64 * waves, kernels(d)


def test_frontier_waves(exe):
    """Four wavefronts to a request's frontier in batches of up to 1,024."""
    _, a, b = talk(exe, "build p 0 100000", "batch p 4 1024", "batch p 4 1025")
    assert kernels(a)[0] == ("k_tile_frontier<4>", 1024, 256)
    assert kernels(b)[0] == ("k_tile_frontier<1>", 257, 256)
