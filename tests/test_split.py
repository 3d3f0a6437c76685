"""Host arithmetic of launches, no GPU needed: how key tiles are shared out among workgroups, which keys are loaded past the
last-level cache, where a short context is compacted."""
import random
import subprocess

from test_bound import _client


def _shares(tmp_path_factory, queries):
    out = subprocess.run([_client(tmp_path_factory, "split_client")], input="".join("%d %d %d %d %d\n" % q for q in queries),
                         check=True, capture_output=True, text=True).stdout
    return [tuple(int(x) for x in line.split()) for line in out.splitlines()]


def test_key_tiles_of_a_launch(tmp_path_factory):
    """Every tile is taken once, pass 2 walks a share backwards over the same tiles, and no share is longer than the first-placed
    workgroups' weighted part of the tiles, rounded up (equal parts where a unit holds one workgroup, or more than two)."""
    rng, n_cu = random.Random(1), 256
    queries = [(8, 64, 194, n_cu, 0), (8, 64, 258, n_cu, 0), (8, 64, 386, n_cu, 0), (4, 128, 770, n_cu, 0), (2, 192, 328, n_cu, 0)]
    while len(queries) < 4000:
        Hk = rng.choice([1, 2, 3, 4, 7, 8, 8, 16, 40, 64, 300])
        n_chunks = rng.randint(1, min(256, max(1, 4 * n_cu // Hk)))
        queries.append((Hk, n_chunks, n_chunks + rng.choice([0, 1, rng.randint(0, 2 * n_chunks), rng.randint(0, 40 * n_chunks)]),
                        n_cu, rng.randint(0, 1)))
    weighted = 0
    for (Hk, n_chunks, n_tiles, _, two), (ok, longest, w) in zip(queries, _shares(tmp_path_factory, queries)):
        assert ok, (Hk, n_chunks, n_tiles, two)
        equal = -(-n_tiles // n_chunks)
        if n_cu < n_chunks * Hk <= 2 * n_cu:
            first = max(1, n_cu // Hk)
            most = -(-n_tiles * w // (w * first + (2048 - w) * (n_chunks - first)))
            weighted += longest > equal
            assert longest <= max(most, equal), (Hk, n_chunks, n_tiles, two, longest, most)
        else:
            assert longest == equal, (Hk, n_chunks, n_tiles, two)
    assert weighted > 100                              # the unequal shares are there


def test_keys_that_are_read_again_stay_in_the_cache(tmp_path_factory):
    """Past the last-level cache go keys of 80 MB that a call reads once and of 112 MB that it reads again, by the other pass or the
    next group of rows; never those that several heads share."""
    mb = 1 << 20
    ask = [(80 * mb, 1, 0), (80 * mb - 1, 1, 0), (112 * mb - 1, 2, 0), (112 * mb, 2, 0), (100 * mb, 4, 0), (400 * mb, 3, 0),
           (80 * mb, 1, 1), (4000 * mb, 1, 1), (4000 * mb, 2, 1)]
    out = subprocess.run([_client(tmp_path_factory, "stream_client")], input="".join("%d %d %d\n" % q for q in ask),
                         check=True, capture_output=True, text=True).stdout
    assert [int(x) for x in out.split()] == [1, 0, 0, 1, 0, 1, 0, 0, 0]


def test_compaction_of_few_heads_has_a_launch_of_its_own(tmp_path_factory):
    """Beside the selection only what one die's units take at once, or heads that spread over the dies."""
    ask = [(1, 32), (1, 33), (1, 36), (4, 32), (4, 34), (5, 1000), (8, 1000), (9, 16), (9, 17), (16, 1000), (17, 1000)]
    out = subprocess.run([_client(tmp_path_factory, "short_client")], input="".join("%d %d\n" % q for q in ask),
                         check=True, capture_output=True, text=True).stdout
    assert [int(x) for x in out.split()] == [1, 0, 0, 1, 0, 1, 1, 1, 0, 1, 1]
