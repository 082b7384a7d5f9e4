"""Counter summaries tell kernels apart whose names begin alike, and the digest
that a stored traffic figure is valid for covers every header that the pair
kernel's unit includes."""
import pathlib
import re
import sqlite3

import pytest

from paper_2603_22274_amd import profiling

CSRC = pathlib.Path(profiling.__file__).resolve().parent / 'csrc'


def _counters(tmp_path, rows):
    d = tmp_path / 'pmc'
    d.mkdir()
    con = sqlite3.connect(str(d / 'run_results.db'))
    con.execute("create table counters_collection (kernel_name text, grid_size integer, counter_name text, "
                "value real)")
    con.executemany("insert into counters_collection values (?, ?, ?, ?)", rows)
    con.commit()
    con.close()
    return str(d)


def test_a_name_is_not_taken_for_a_longer_one(tmp_path):
    ns = 'felis::(anonymous namespace)::'
    d = _counters(tmp_path, [(f"{ns}k_spread(felis::LegDev const*)", 9216, "SQ_WAVES", 10.0),
                             (f"{ns}k_spread_wide(felis::LegDev const*)", 9216, "SQ_WAVES", 30.0),
                             (f"{ns}k_ukn_spread(felis::LegDev const*)", 99999, "SQ_WAVES", 70.0),
                             (f"void {ns}k_pairs<0>(felis::LegDev const*)", 512, "SQ_WAVES", 5.0),
                             (f"void {ns}k_build<1>(felis::LegDev const*)", 64, "SQ_WAVES", 2.0)])
    c = profiling.counters(d, ['k_spread', 'k_spread_wide', 'k_pairs<0>', 'k_build'])
    assert {k: v['SQ_WAVES'] for k, v in c.items()} == pytest.approx(
        {'k_spread': 10.0, 'k_spread_wide': 30.0, 'k_pairs<0>': 5.0, 'k_build': 2.0})
    assert profiling._counter(profiling._db(d), 'k_spread') == (10.0, 1)
    assert profiling._counter(profiling._db(d), 'k_spread_wide') == (30.0, 1)
    assert profiling._counter(profiling._db(d), 'k_gather') == (None, 0)


def test_the_digest_covers_the_pair_kernels_headers():
    inc = re.findall(r'#include "([^"]+)"', (CSRC / 'nonbonded.hip').read_text())
    assert set(inc) | {'nonbonded.hip'} <= set(profiling.PAIR_SOURCES)
    assert all((CSRC / f).is_file() for f in profiling.PAIR_SOURCES)
