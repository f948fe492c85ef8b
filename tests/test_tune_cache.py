"""The file of the tuner's table (BTC_TUNE_CACHE) across its formats: host
state only."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """import sys; sys.path.insert(0, %r)
from paper_2601_03754_amd import btc
for a in sys.argv[1:]:
    v = [int(x) for x in a.split(",")]
    if len(v) == 5:
        btc.btc_tune_set(*v)
    elif len(v) == 3:
        print(*btc.btc_select_strategy(*v))
    else:
        print(btc.btc_tune_get(*v))
""" % ROOT


def run(cache, *calls):
    r = subprocess.run([sys.executable, "-c", CODE, *calls], env=dict(os.environ, BTC_TUNE_CACHE=str(cache)),
                       check=True, capture_output=True, text=True)
    return r.stdout.split()


def test_files_without_a_format_line(tmp_path):
    """The factor's variants at padded size 64 have had both numberings in
    files without a format line: such a line is ignored (the default stays),
    every other line is read."""
    cache = tmp_path / "tune.txt"
    cache.write_text("v 0 0 64 0 0\nv 0 0 64 1 0\nv 0 1 64 0 0\nv 0 0 32 1 2\nv 6 1 96 0 2\ns 0 16 8 1 2\n")
    got = run(cache, "0,0,64,0", "0,0,40,3", "0,1,50,0", "0,0,24,1", "6,1,90,0", "16,8,0")
    assert got == ["1", "1", "1", "2", "2", "1", "2"]


def test_written_files_keep_every_key(tmp_path):
    cache = tmp_path / "tune.txt"
    run(cache, "0,0,64,0,0", "0,2,40,3,0", "0,0,24,1,1", "6,0,64,0,1")
    assert cache.read_text().startswith("f 2\n")
    assert run(cache, "0,0,33,0", "0,0,33,1", "0,2,64,1", "0,0,17,9", "6,0,50,0") == ["0", "1", "0", "1", "1"]


def test_files_of_a_later_format(tmp_path):
    cache = tmp_path / "tune.txt"
    cache.write_text("f 3\nv 0 0 32 1 2\n")
    assert run(cache, "0,0,24,1") == ["0"]
