"""The weight-streaming kernel's activation ring in LDS, replayed on the host: between two barriers no wavefront may write what another one reads
or writes.  The wavefronts' program order is that of pair_of_tiles in gemm_stream_body.h; the stage of the epilogue comes from stream_stages.h,
compiled here."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_04667_amd", "csrc")
WAVES = 8


@pytest.fixture(scope="module")
def epilogue_stage(tmp_path_factory):
    d = tmp_path_factory.mktemp("stages")
    (d / "t.cpp").write_text('#include <cstdio>\n#include "stream_stages.h"\nint main() { for (int s = 2; s <= 3; ++s) for (int a = 0; a < s; ++a) '
                             'for (int l = 0; l < 2; ++l) std::printf("%d %d %d %d\\n", s, a, l, moe::stream_epilogue_stage(s, a, l != 0)); }\n')
    cxx = shutil.which("g++") or shutil.which("c++") or "/opt/rocm/bin/amdclang++"
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t")], check=True)
    rows = [tuple(map(int, l.split())) for l in subprocess.run([str(d / "t")], check=True, capture_output=True, text=True).stdout.splitlines()]
    table = {(s, a, bool(l)): e for s, a, l, e in rows}
    return lambda stages, sa, last: table[stages, sa, last]


def accesses(large, tasks, pairs, stage_of_epilogue):
    """(barriers passed at the beginning, at the end; "read" or "write"; wavefront; stage; which 2 KB of it) of all wavefronts, for a stream of
    `tasks` tiles of `pairs` pairs of K-tiles each: `large` 256-row tiles with three stages, else 128-row ones with two."""
    out = []
    stages, total = (3 if large else 2), tasks * pairs
    for wave in range(WAVES):
        # a wavefront copies 32 or 16 rows of 128 bytes and reads half of the tile's rows (of the small tile 16 of every 32)
        own = (2 * wave, 2 * wave + 1) if large else (wave,)
        readable = range(wave // 4 * 8, wave // 4 * 8 + 8) if large else range(wave // 4, 8, 2)
        epoch, flights = 0, []                              # copies in flight: (epoch of the request, stage, pair of K-tiles)

        def request(pair):
            if pair < total:
                flights.append((epoch, pair % stages, pair))

        def read(stage):
            out.extend((epoch, epoch, "read", wave, stage, r) for r in readable)

        def barrier(landed):                                # everything of the pairs up to `landed` has arrived
            nonlocal epoch
            epoch += 1
            for f in [f for f in flights if f[2] <= landed]:
                out.extend((f[0], epoch - 1, "write", wave, f[1], r) for r in own)
                flights.remove(f)

        request(0)
        request(1)
        barrier(0)
        read(0)                                             # first rows of the first tile
        for q in range(total):
            sa, last, steady = q % stages, q == total - 1, q < total - 2
            if large:
                read(sa)                                    # second half of the even tile's rows
                if steady:
                    request(q + 2)
            barrier(q if steady else total)
            read(sa)                                        # first rows of the odd tile, and the rest of them
            read(sa)
            if not last:
                barrier(q + 1 if steady else total)
                if not large and steady:
                    request(q + 2)
                read((q + 1) % stages)                      # first rows of the next pair
            if (q + 1) % pairs == 0:                        # 4 KB to a wavefront
                out.extend((epoch, epoch, "write", wave, stage_of_epilogue(stages, sa, last), r) for r in (2 * wave, 2 * wave + 1))
        for f in flights:
            out.extend((f[0], epoch, "write", wave, f[1], r) for r in own)
    return out


def conflicts(ops):
    by_place = {}
    for op in ops:
        by_place.setdefault(op[4:], []).append(op)
    return [(a, b) for place in by_place.values() for a in place if a[2] == "write" for b in place
            if a[3] != b[3] and max(a[0], b[0]) <= min(a[1], b[1])]


@pytest.mark.parametrize("tasks,pairs", [(1, 3), (1, 4), (1, 5), (2, 3), (2, 4), (3, 5), (4, 32)])
@pytest.mark.parametrize("large", [True, False])
def test_no_wavefront_writes_rows_that_another_still_reads(epilogue_stage, large, tasks, pairs):
    assert not conflicts(accesses(large, tasks, pairs, epilogue_stage))


@pytest.mark.parametrize("tasks,pairs", [(1, 3), (2, 4), (3, 5)])
def test_the_replay_notices_a_stage_that_is_still_read(tasks, pairs):
    # the pair's own stage at the end of the stream, where no barrier follows the last reads; and the next pair's before it
    assert conflicts(accesses(True, tasks, pairs, lambda stages, sa, last: sa))
    if tasks > 1:
        assert conflicts(accesses(True, tasks, pairs, lambda stages, sa, last: (sa + 1) % stages))
