"""Host arithmetic of the library's headers, no GPU needed: the top-k's bound leaves the candidate buffers room, the sample
is scattered, attributes are set once per device."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _client(tmp_path_factory, name):
    gxx = shutil.which("g++")
    assert gxx, "g++ is part of the toolchain this repository builds with"
    exe = str(tmp_path_factory.mktemp("bound") / name)
    subprocess.run([gxx, "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(ROOT, "paper_2601_07667_amd", "csrc"),
                    os.path.join(ROOT, "tests", name + ".cpp"), "-o", exe], check=True)
    return exe


@pytest.fixture(scope="module")
def bound(tmp_path_factory):
    exe = _client(tmp_path_factory, "bound_client")

    def ask(queries):
        out = subprocess.run([exe], input="".join("%d %d %d\n" % q for q in queries), check=True, capture_output=True, text=True).stdout
        return [tuple(int(x) for x in ln.split()) for ln in out.splitlines()]
    return ask


def test_slack_stays_within_the_candidate_buffers(bound):
    """Wherever the bound may pass more than the m-th sample key, the tokens that m + slack sample keys stand for fit a
    row's buffer with 3 standard deviations of the m-th key's count to spare, and a tile's segment with 4; or the m-th
    key alone overflows one of them by a deviation."""
    queries = [(T, k, runs) for T in (12289, 16352, 20001, 24544, 32736, 65504, 131040, 262080, 1048544)
               for k in (1, 64, 500, 2016, 3000, 4000, 4540, 5250, 5730, 6540, 6990, 8160, 9000, 9090, 10000, 11440, 11800, 12600, 14000)
               for runs in (0, 1) if k <= T]
    used = full = 0
    for (T, k, runs), (n_s, run, m, slack, cap, tile, seg) in zip(queries, bound(queries)):
        assert 0 <= slack <= m // 8, (T, k, runs)
        if slack == 0:
            continue
        row_dev, tile_dev = T / n_s * (run * m) ** 0.5, ((tile / n_s) ** 2 * run * m + 2 * tile) ** 0.5
        if m * T / n_s > cap + row_dev * (1 - 1e-5) or m * tile / n_s > seg + tile_dev * (1 - 1e-5):
            continue
        used += 1
        full += slack == m // 8
        assert (m + slack) * T / n_s + 3 * row_dev <= cap * (1 + 1e-6), (T, k, runs)
        assert (m + slack) * tile / n_s + 4 * tile_dev <= seg * (1 + 1e-6), (T, k, runs)
    assert used > 100 and full > 80                    # the early stop is still there for ordinary budgets


def test_ordinary_budgets_keep_the_whole_slack(bound):
    queries = [(T, 2016, runs) for T in (32736, 131040, 262080) for runs in (0, 1)]
    for q, (n_s, run, m, slack, *_) in zip(queries, bound(queries)):
        assert slack == m // 8 > 0, q


def test_candidates_of_pooled_scores(tmp_path_factory):
    """Half the candidate buffer is made room for only where the bound admits more once in 10^6 rows, also where pooling makes
    neighbouring sampled keys alike (the variance of what it admits is then as many times the independent keys')."""
    queries = [(T, k, S) for T in (12289, 20001, 32736, 65504, 131040, 262080, 1048544) for k in (64, 1000, 2016, 2500, 3000, 3500, 4064)
               for S in (1, 7, 31, 63, 129)]
    out = subprocess.run([_client(tmp_path_factory, "cap_client")], input="".join("%d %d %d\n" % q for q in queries), check=True,
                         capture_output=True, text=True).stdout
    halves = narrowed = 0
    for (T, k, S), line in zip(queries, out.splitlines()):
        n_s, m, slack, alike, cap = (int(x) for x in line.split())
        assert alike == -(-S // (T // n_s))
        admits, dev = (m + slack) * T / n_s, T / n_s * m ** 0.5
        assert cap == 16384 or (cap == 8192 and admits + 5 * alike ** 0.5 * dev <= 8192 * (1 + 1e-6)), (T, k, S)
        halves += cap == 8192
        narrowed += cap == 16384 and admits + 5 * dev <= 8192
    assert halves > 80 and narrowed > 0                # the ordinary budgets; the widest poolings


def test_sample_positions(tmp_path_factory):
    """One position in every stride of the row up to its last few tokens, and for every period up to 64 (and some
    longer ones) every phase of it about as often as any other: between half and twice, with six deviations to spare."""
    sizes = (12289, 16352, 32736, 32769, 65504, 131040, 131072, 262080, 262145, 500001, 1048544, 2097152)
    out = subprocess.run([_client(tmp_path_factory, "sample_client")], input="\n".join(map(str, sizes)), check=True,
                         capture_output=True, text=True).stdout
    for T, line in zip(sizes, out.splitlines()):
        stride, *pos = (int(x) for x in line.split())
        assert 900 <= len(pos) <= 8192 and T - stride < len(pos) * stride <= T
        assert all(j * stride <= p < (j + 1) * stride for j, p in enumerate(pos)), T
        for period in [*range(2, min(65, stride + 1)), 96, 128]:
            count, mean = [0] * period, len(pos) / period
            for p in pos:
                count[p % period] += 1
            if stride >= period:
                assert min(count) >= mean / 2 - 6 * mean ** 0.5 and min(count) > 0, (T, period)
                assert max(count) <= 2 * mean + 6 * mean ** 0.5, (T, period)


def test_once_per_device(tmp_path_factory):
    """Kernel attributes are set on every device that launches the kernel, not once in the process; failures are tried again."""
    out = subprocess.run([_client(tmp_path_factory, "once_client")], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout == "ok\n"
