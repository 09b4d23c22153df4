"""The rules of the default schedules, asked of the library on the CPU (a small
program linked with it): what a pack, a copy or a sum of a given shape gets."""
import os
import subprocess

import pytest

from paper_2309_07337_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
FIELDS = ("tile_rows", "block_threads", "blocks_per_cu", "nontemporal", "unroll", "push_pack", "lds_window", "pair_rows")
GATHER, SUM = 0, 1
PACK, REDIST, UNPACK, BWD = range(4)
CUS = 256       # without a device


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if not os.path.exists(B.HIPCC):
        pytest.skip("hipcc not installed")
    if not os.path.exists(B.LIB):
        B.build_library()
    exe = str(tmp_path_factory.mktemp("sched") / "default_sched")
    r = subprocess.run([B.HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", B.INCLUDE, "-I", B.CSRC,
                        os.path.join(HERE, "sched", "default_sched.cpp"), "-o", exe,
                        "-L", os.path.dirname(B.LIB), "-l:" + os.path.basename(B.LIB),
                        "-Wl,-rpath," + os.path.dirname(B.LIB)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[:4000]

    def ask(kind, row_bytes, phase, rows, owned=0, runs=1, terms=0, values=1, jobs=1, nbytes=None, source=0, identity=0,
            fresh=0):
        line = [kind, row_bytes, phase, rows, owned, runs, terms, values, jobs,
                2 * rows * row_bytes if nbytes is None else nbytes, source, identity, fresh]
        out = subprocess.run([exe], input=" ".join(map(str, line)), capture_output=True, text=True, check=True).stdout
        return dict(zip(FIELDS, map(int, out.split())))
    return ask


@pytest.mark.parametrize("row_bytes", [4, 8, 12, 16, 24, 40, 56])
@pytest.mark.parametrize("n", [2_000_000, 8_000_000])
def test_packs_of_short_rows(rules, row_bytes, n):
    """Pushed where at least half as many rows are packed as the source has: a
    push walks every one of them."""
    packed = lambda rows: rules(GATHER, row_bytes, PACK, rows, owned=n, runs=26, source=n * row_bytes)["push_pack"]
    assert n * row_bytes > 4 << 20
    assert packed(n // 33) == 0 and packed(n // 4) == 0 and packed(n // 2 - 1) == 0
    assert packed(n // 2) == 1 and packed(n) == 1 and packed(3 * n) == 1
    assert rules(GATHER, row_bytes, PACK, 3000, owned=1000, source=1000 * row_bytes)["push_pack"] == 0


@pytest.mark.parametrize("row_bytes", [4, 8, 12, 24, 40, 56])
def test_lists_in_no_order(rules, row_bytes):
    """Short rows in no order are pulled where the packed rows are beyond the
    Infinity Cache; in messages of ascending rows, or fewer, they are pushed."""
    def push(rows, run):
        return rules(GATHER, row_bytes, PACK, rows, owned=rows, runs=rows // run, source=rows * row_bytes)["push_pack"]

    small, large = (150 << 20) // row_bytes, (250 << 20) // row_bytes
    assert push(small, 1) == 1 and push(small, 4096) == 1
    assert push(large, 1) == 0 and push(large, 64) == 0
    assert push(large, 4096) == 1
    # (what a batch packs is spread over its jobs)
    assert rules(GATHER, row_bytes, PACK, large, owned=large, runs=large, jobs=20,
                 source=large * row_bytes // 20)["push_pack"] == 1
    assert rules(GATHER, 64, PACK, large, owned=large, runs=large, source=large * 64)["push_pack"] == 1


@pytest.mark.parametrize("row_bytes", [64, 128, 256, 800])
def test_pushed_tiles_cover_the_source(rules, row_bytes):
    """Their size follows the rows they walk: few rows packed from many make no
    more tiles than many do, and a small source still gives every CU two."""
    def tile(rows, owned):
        s = rules(GATHER, row_bytes, PACK, rows, owned=owned, source=owned * row_bytes, fresh=1)
        assert s["push_pack"] == 1
        return s["tile_rows"]

    n = 1_000_000
    dense = tile(n, n)
    assert all(tile(n // k, n) >= dense for k in (2, 4, 16, 64, 1000))
    least = max(16, 4096 // row_bytes)
    for rows in (100, 3000):
        assert 3000 // tile(rows, 3000) >= min(2 * CUS, 3000 // least)


STAGE_ROWS, WIN_BYTES = 512, 72 << 10     # rows whose pointers a sum's tile stages; its largest window


@pytest.mark.parametrize("terms_per_row", [0, 1, 5, 8, 40])
@pytest.mark.parametrize("rows", [100, 20_000, 3_000_000])
@pytest.mark.parametrize("jobs", [1, 40, 1000])
@pytest.mark.parametrize("fresh", [0, 1])
def test_sums_of_two_single_values(rules, terms_per_row, rows, jobs, fresh):
    """Rows of two FP32 values are no one-value rows: their sums stage their
    pointers (unless hardly one has a term), or read a window that fits, and
    never go one row a lane."""
    terms = rows * terms_per_row
    for source in (terms * 8 // jobs, WIN_BYTES, 4 << 20):
        s = rules(SUM, 8, BWD, rows, terms=terms, values=2, jobs=jobs, nbytes=(rows + terms) * 12, source=source,
                  fresh=fresh)
        assert s["pair_rows"] == 0
        assert s["tile_rows"] <= STAGE_ROWS or (s["lds_window"] == 1 and source <= WIN_BYTES) or 8 * terms <= rows
    one = rules(SUM, 8, BWD, rows, terms=terms, values=1, jobs=jobs, source=1 << 20)
    assert one["pair_rows"] == 1


@pytest.mark.parametrize("rows_a_job,lanes", [(1, 256), (100, 256), (128, 256), (129, 512), (1000, 512)])
def test_windows_of_few_rows(rules, rows_a_job, lanes):
    """A window's sums run a lane a row: no 512 lanes for jobs of fewer rows."""
    jobs, terms = 6000, 8 * rows_a_job
    s = rules(SUM, 8, BWD, jobs * rows_a_job, terms=jobs * terms, values=2, jobs=jobs, source=8 * terms)
    assert (s["lds_window"], s["block_threads"]) == (1, lanes)


@pytest.mark.parametrize("row_bytes", [64, 100, 400, 2048])
def test_long_rows_packed_by_halves(rules, row_bytes):
    """A request that packs at most half of its long rows pulls them; a world's
    push copies a caller's rows, so it stays; longer rows are pushed too."""
    def push(rows, rb=row_bytes, **kw):
        return rules(GATHER, rb, PACK, rows, owned=100_000, source=100_000 * rb, **kw)["push_pack"]

    assert push(50_000) == 0 and push(10) == 0 and push(50_001) == 1 and push(300_000) == 1
    assert push(10, fresh=1) == 1 and push(10, rb=2052) == 1


@pytest.mark.parametrize("row_bytes", [4, 8, 12, 24, 56])
def test_messages_of_every_fourth_row(rules, row_bytes):
    """Dense messages of short rows are pulled, unless longer ones are read several times."""
    n = 8_000_000
    def push(rows, runs):
        return rules(GATHER, row_bytes, PACK, rows, owned=n, runs=runs, source=n * row_bytes)["push_pack"]

    assert push(n, 4) == 0 and push(n, 5) == 1
    assert push(3 * n, 12) == (0 if row_bytes <= 8 else 1) and push(3 * n, 13) == 1


@pytest.mark.parametrize("row_bytes", [64, 100, 256, 1024, 1028, 2048, 2052, 10_000])
@pytest.mark.parametrize("jobs", [1, 1000])
@pytest.mark.parametrize("fresh", [0, 1])
@pytest.mark.parametrize("terms_per_row", [0, 1, 3, 4, 8, 40])
def test_sums_of_few_long_rows(rules, row_bytes, jobs, fresh, terms_per_row):
    """512 lanes and a tile for every CU where the rows are short for their
    terms, with no more terms in it than a tile stages; a world's ranks are one job."""
    rows = 4 * CUS
    s = rules(SUM, row_bytes, BWD, rows, terms=terms_per_row * rows, jobs=jobs, nbytes=1 << 20, source=1 << 16,
              fresh=fresh)
    shrunk = jobs == 1 or fresh == 1
    assert (s["block_threads"] == 512) == (shrunk and row_bytes <= (2048 if terms_per_row <= 3 else 1024))
    assert (s["tile_rows"] < 64) == shrunk
    large = rules(SUM, 64, BWD, 260_000, terms=260_000 * terms_per_row, source=1 << 24)
    assert large["block_threads"] == 512 and large["tile_rows"] * terms_per_row <= 2048


@pytest.mark.parametrize("row_bytes", [64, 100, 2000, 2004])
def test_lanes_of_pushed_long_rows(rules, row_bytes):
    """256 for rows of a power of two, and for a request's others of up to 2 KiB
    that are packed at most three times."""
    def lanes(rows, **kw):
        return rules(GATHER, row_bytes, PACK, rows, owned=100_000, source=100_000 * row_bytes, **kw)["block_threads"]

    assert lanes(100_000) == lanes(300_000) == 256
    assert lanes(300_001) == lanes(300_000, fresh=1) == (256 if row_bytes == 64 else 512)
