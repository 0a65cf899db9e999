"""Host check of the split of a visit list's arrival query into chunks of visits
(not a GPU test): the chunk length is a multiple of 256, never shrinks as the list
grows and keeps a list at 32 chunks, read off the number of work items launched."""
import fake_hip

CODE = r"""
def items(n, K):  # tile t sees the chunks that start before its last visit does
    return sum((min(n, p + 256) - 2) // K + 1 if min(n, p + 256) > 1 else 0 for p in range(0, n, 256))
lengths = []
for n in (300, 4096, 16384, 20000, 24576, 24577, 25600, 26367, 26368, 28224, 32768, 65536):
    t = np.arange(n) * 1e-6
    v = dd.Visits(np.zeros(n), np.zeros(n), t, np.full(n, 1e-6))
    out = buf(n)
    launches()
    ok(lib.dd_visits_arrival(v._h, 0, ptr(out), 1, None))
    got = [x for name, x, _ in launches() if "k_visit_arrival" in name]
    assert len(got) == 1, got
    fit = [K for K in range(256, 4097, 256) if items(n, K) == got[0]]
    assert fit, (n, got)
    lengths.append((n, fit[0], fit[-1]))
    assert -(-n // fit[-1]) <= 32, lengths
for (n0, _, hi0), (n1, lo1, hi1) in zip(lengths, lengths[1:]):
    lo0 = [lo for n, lo, _ in lengths if n == n0][0]
    assert hi1 >= lo0, lengths
print(lengths)
"""


def test_chunk_lengths(tmp_path):
    fake_hip.run(tmp_path, CODE)
