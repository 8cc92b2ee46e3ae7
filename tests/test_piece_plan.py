"""The plan and scan arithmetic of the piece partition, run on the host
(tests/piece_plan_driver.cpp over csrc/piece_plan.h): the array sizes and LDS
limits that the kernels rely on hold for the groups that sequences make, at the
key lengths and load factors where they are closest. Whole numbers: there is no
tolerance."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("needs hipcc")
    exe = str(tmp_path_factory.mktemp("plan") / "driver")
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-O2", "-std=c++17",
                    os.path.join(ROOT, "tests", "piece_plan_driver.cpp"), "-o", exe], check=True, capture_output=True)

    def run(*args):
        out = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True, timeout=300).stdout
        words = out.split()[1:]
        return dict(zip(words[::2], map(int, words[1::2])))

    return run


# One sequence (the most pieces for its k-mers) and reads at 30x; long keys with
# many k-mers per slot are cut by their bases, into several times the sub-tables
# that their k-mers would make.
@pytest.mark.parametrize("k,m,load,block,n_bins,G,cov,read", [
    (479, 11, 4.0, 0, 1, 11_500_000, 0, 0), (479, 11, 4.0, 0, 1, 6_000_000, 0, 0), (479, 11, 0.0, 0, 1, 11_500_000, 0, 0),
    (300, 9, 4.0, 0, 3, 6_000_000, 0, 0), (256, 11, 4.0, 1024, 1, 8_000_000, 0, 0), (200, 11, 4.0, 512, 2, 8_000_000, 0, 0),
    (200, 11, 0.0, 0, 1, 1_000_000, 30, 1000), (99, 9, 4.0, 0, 1, 500_000, 30, 250), (65, 9, 0.0, 512, 1, 500_000, 30, 150),
    (65, 9, 0.05, 0, 4, 1_000_000, 10, 150), (28, 9, 4.0, 0, 1, 500_000, 30, 100), (20, 7, 0.0, 0, 2, 500_000, 30, 100)])
def test_sub_tables_fit_their_arrays(driver, k, m, load, block, n_bins, G, cov, read):
    r = driver("genome", k, m, load, block, n_bins, G, cov, read, k + n_bins)
    assert r["groups"] <= r["grp_cap"]
    assert r["tables"] <= r["tab_cap"] and r["failed"] == 0
    assert r["pieces"] <= r["list"]
    assert r["most_halves"] <= r["max_halves"]
    assert r["lost"] == 0


# 2^18 groups, the most a bin has: their weights add up to under and over 2^32
@pytest.mark.parametrize("k,load,kmers,pieces", [(65, 0.005, 200, 20), (65, 0.005, 300, 30), (28, 0.005, 2_000, 500),
                                                 (479, 0.01, 250, 12), (65, 0.0, 6_000, 300)])
def test_weights_of_a_very_large_bin(driver, k, load, kmers, pieces):
    """Every sub-table is one run of groups, of no more k-mers than a unit of weight and half a group to either side."""
    r = driver("groups", k, 9, load, 0, 1 << 18, kmers, pieces)
    assert r["heavy"] == 0 and r["failed"] == 0
    assert r["lost"] == 0
    assert r["tables"] <= r["tab_cap"]
    assert r["most_halves"] <= r["max_halves"]
    assert r["most_kmers"] <= max(2 * kmers, 2 * r["kmers"] // r["tables"] + kmers)


@pytest.mark.parametrize("kmers", [(1 << 32) - 1, 1 << 32, (1 << 32) + 5, 9_000_000_000])
@pytest.mark.parametrize("groups", [1, 3])
def test_k_mers_of_a_group_stay_in_their_half_word(driver, kmers, groups):
    """One sub-minimizer can bring all of a bin's k-mers: either the groups' counts hold them, or the bin is left whole."""
    r = driver("groups", 65, 9, 0.0, 0, groups, kmers, kmers // 48)
    if r["failed"] == 0:
        assert r["pieces"] == groups * (kmers // 48)
        assert r["heavy"] == groups and r["heavy_kmers"] == groups * kmers


@pytest.mark.parametrize("load", [0.0, 0.3, 4.0])
@pytest.mark.parametrize("k,block", [(20, 0), (28, 512), (65, 0), (99, 0), (200, 512), (256, 0), (479, 0)])
def test_bases_of_a_sub_table_fit_the_stage(driver, k, block, load):
    """Whatever the sizes of a bin's groups, large ones side by side among them, a sub-table's bases fit its LDS stage."""
    r = driver("random", k, load, block, k)
    assert r["failed"] == 0 and r["lost"] == 0
    assert 0.8 * r["max_halves"] < r["most_halves"] <= r["max_halves"]


@pytest.mark.parametrize("k,m,n_bins,G,cov,read", [
    (20, 7, 2, 2_000_000, 0, 0), (28, 9, 4, 2_000_000, 0, 0), (55, 9, 2, 500_000, 10, 150), (65, 9, 1, 2_000_000, 0, 0),
    (99, 9, 4, 500_000, 10, 250), (111, 9, 1, 2_000_000, 0, 0), (200, 11, 1, 2_000_000, 0, 0), (300, 7, 2, 2_000_000, 0, 0),
    (479, 11, 1, 4_000_000, 0, 0), (480, 15, 1, 2_000_000, 0, 0)])
def test_expected_pieces(driver, k, m, n_bins, G, cov, read):
    """The plan's estimate counts every kind of cut. It is an upper one: a tenth is added for change of sub-minimizers
    and ends, and turns shared out evenly are a few less; it is never short by more than 5 %."""
    r = driver("genome", k, m, 0.0, 0, n_bins, G, cov, read, k)
    assert r["pieces"] / 1.05 <= r["expected"] <= 1.3 * r["pieces"]


@pytest.mark.parametrize("load,n_bins,G", [(0.0, 1, 11_500_000), (0.0, 1, 7_000_000), (4.0, 1, 18_000_000), (0.0, 4, 18_000_000)])
def test_groups_of_long_keys_are_seldom_heavy(driver, load, n_bins, G):
    """Keys above 256 bases whose groups are heavy are counted in HBM tables: a random sequence leaves next to none."""
    r = driver("genome", 479, 11, load, 0, n_bins, G, 0, 0, 1)
    assert r["heavy_kmers"] <= 0.01 * r["kmers"]
