"""The host side of the library's calls, on a HIP runtime that runs nothing
(tests/fake_hip.c): what a call allocates and launches, and what is left when
an allocation or a launch is refused.  Each test's script runs in a process of
its own, in which that runtime is loaded first."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, json, random, sys
sys.path.insert(0, sys.argv[2])
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
fake.fake_log.restype = ctypes.c_char_p
import paper_2505_12976_amd as sz
lib = sz.load_library()
U16, I32, FAR = sz.U16, sz.I32, 1 << 46   # FAR: some device address, never read
def context():
    h = ctypes.c_void_p()
    fake.fake_reset()
    assert lib.schulze_create(ctypes.byref(h), 0) == 0
    fake.fake_reset()
    return h
def log():
    return fake.fake_log().decode().splitlines()
def launched():
    return [l.split()[1] for l in log() if l.split()[0] in ("launch", "cooperative")]
def out(x):
    print(json.dumps(x))
"""


@pytest.fixture(scope="session")
def fake_hip(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake_hip") / "libfake_hip.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "fake_hip.c"), "-o", so], check=True, capture_output=True)

    def run(script):
        r = subprocess.run([sys.executable, "-c", PRELUDE + script, so, ROOT], capture_output=True, text=True,
                           timeout=300)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout.splitlines()[-1])

    return run


TRAIN = """
net = sz.MlpState(FAR, FAR, FAR, FAR, FAR, 1e-3, 0.9, 0.999, 1e-8)
batch = sz.TrainBatch(FAR, FAR, FAR, 5000, 40)
def step(h):
    return lib.schulze_mlp_train_step(h, None, ctypes.byref(net), ctypes.byref(batch), FAR)
"""


def test_train_step_that_fails_leaves_nothing_queued(fake_hip):
    """A refused allocation (each in turn) or kernel attribute is found before
    the first launch, so that the step counter stands still."""
    got = fake_hip(TRAIN + """
rows = []
h = context()
assert step(h) == 0
allocations = sum(l.startswith("malloc") for l in log())
for k in range(allocations):
    h = context()
    fake.fake_fail_malloc(k)
    rows.append([step(h), launched()])
h = context()
fake.fake_fail_attribute(1)
rows.append([step(h), launched()])
out([allocations, rows])
""")
    allocations, rows = got
    assert allocations >= 3
    for rc, launches in rows[:-1]:
        assert rc == -3 and launches == []
    assert rows[-1] == [-4, []]


def test_loss_takes_as_many_elections_as_wavefronts(fake_hip):
    """64 threads per election beyond the few that get a workgroup each: up to
    2^26 - 4 elections fit one launch."""
    got = fake_hip("""
rows = []
for E in (1, 1024, 1025, 1 << 24, (1 << 26) - 4):
    h = context()
    rc = lib.schulze_mlp_loss(h, None, FAR, FAR, FAR, E, FAR, FAR)
    rows.append([E, rc, log()[-1]])
out(rows)
""")
    for E, rc, line in got:
        assert rc == 0, (E, line)
        many = E > 1024
        assert ("k_seg_loss_many" in line) == many
        assert int(line.split()[2]) == (-(-E // 4) if many else E)


def test_smaller_counts_allocate_nothing(fake_hip):
    """A context that has made a count makes every smaller one of its kind (fewer
    voters, shorter ballots, fewer candidates; with voter weights or without,
    with room for full rankings or without) without a new allocation, whatever
    kernels the smaller call takes: an eager call sizes the workspace for the
    calls that are captured after it."""
    got = fake_hip("""
rng = random.Random(7)
def log_uniform(lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))
def pairwise(h, n, L, m, weighted, ids):
    assert lib.schulze_pairwise(h, None, FAR, ids, n, L, m, FAR if weighted else None, I32, 2 * FAR, m) == 0
bad, routed = [], set()
for trial in range(1000):
    m, n = log_uniform(2, 20000), log_uniform(1, 200000)
    L = m if rng.random() < 0.4 else log_uniform(1, m)
    while n * L > 1 << 27:
        n = max(1, n // 2)
    weighted, ids = rng.random() < 0.4, rng.choice([U16, I32])
    h = context()
    pairwise(h, n, L, m, weighted, ids)
    for smaller in range(12):
        # (LDS rows are wider and workgroups fewer above 16384 candidates)
        m2 = log_uniform(1, m) if m <= 16384 else rng.randint(16385, m)
        if rng.random() < 0.3:
            m2 = max(m2, m - rng.randint(0, 3))
        L2 = min(L, m2) if rng.random() < 0.5 else log_uniform(1, min(L, m2))
        if (L2 >= m2 - 1) != (L >= m - 1):
            if L < m - 1 and m2 < 3:
                continue
            L2 = m2 - 2 if L < m - 1 else min(L, m2)
        n2 = max(1, n - rng.randint(0, 3)) if rng.random() < 0.3 else log_uniform(1, n)
        fake.fake_reset()
        pairwise(h, n2, L2, m2, weighted, ids)
        routed.add(any("k_route" in l for l in launched()))
        if any(l.startswith("malloc") for l in log()):
            bad.append([[n, L, m], [n2, L2, m2], weighted, [l for l in log() if l.startswith("malloc")]])
            break
    lib.schulze_destroy(h)
out([bad, sorted(routed)])
""")
    bad, routed = got
    assert routed == [False, True]
    assert bad == []


def test_smaller_features_allocate_nothing(fake_hip):
    got = fake_hip("""
rng = random.Random(3)
bad = []
def features(h, m):
    assert lib.schulze_features(h, None, FAR, m, m, I32, 0, 1.0, 2 * FAR) == 0
sizes = [1, 63, 64, 65, 700, 3967, 3968, 3969, 4032, 4033, 7872, 7873, 7936, 7937, 8000, 20000, 65535]
for m in sizes + list(range(3900, 8100, 97)):
    h = context()
    features(h, m)
    fake.fake_reset()
    for m2 in [k for k in sizes if k <= m] + [rng.randint(1, m) for _ in range(60)]:
        features(h, m2)
    if any(l.startswith("malloc") for l in log()):
        bad.append([m, [l for l in log() if l.startswith("malloc")]])
    lib.schulze_destroy(h)
out(bad)
""")
    assert got == []


@pytest.mark.parametrize("n,L,m,weighted,one_pass", [
    (1000, 64, 64, False, True), (1400, 20, 1000, False, True), (20000, 25, 389, False, True),
    (20000, 10, 2000, False, False), (300, 20, 4096, False, True), (300, 20, 4097, False, False),
    # short weighted ballots: as many bits of weights as their total allows
    (400, 20, 1000, True, True), (800, 20, 1000, True, False), (1400, 20, 1000, True, False),
    (2000, 25, 389, True, True), (7001, 25, 389, True, True), (12000, 25, 389, True, False),
    (30000, 20, 64, True, True), (100000, 10, 128, True, True), (300, 30, 2000, True, False),
    (64, 50, 4096, True, True), (128, 50, 4096, True, False),
    # long ones: the pairs they can list cost more
    (1400, 1000, 1000, True, True), (3000, 389, 389, True, True), (32, 4096, 4096, True, True),
    (30000, 256, 256, True, True), (40000, 256, 256, True, False), (1, 1, 1, True, True),
])
def test_route_by_size(fake_hip, n, L, m, weighted, one_pass):
    got = fake_hip(f"""
h = context()
assert lib.schulze_pairwise(h, None, FAR, U16, {n}, {L}, {m}, FAR if {weighted} else None, I32, 2 * FAR, {m}) == 0
out([any("k_route" in l for l in launched()), any("k_planes_all" in l or "k_planes_short" in l for l in launched())])
""")
    assert got == [not one_pass, one_pass]


@pytest.mark.parametrize("m,ids,tiles", [(129, "U16", 3), (700, "U16", 11), (6200, "U16", 49), (300, "I32", 5),
                                         (2100, "I32", 17 + 34)])
def test_closure_when_cooperative_launches_are_refused(fake_hip, m, ids, tiles):
    """The phased launches instead, on integers: 16-bit matrices are stored as
    keys before the refusal is known, and go back to values first."""
    got = fake_hip(f"""
h = context()
fake.fake_refuse_cooperative(1)
assert lib.schulze_closure(h, None, FAR, {m}, {m}, {ids}, 0, 2 * FAR, {m}) == 0
out(launched())
""")
    names = [next((k for k in ("k_fw_decode", "k_fw_diag", "k_fw_panel", "k_fw_rest") if k in n), None) for n in got]
    if ids == "U16":
        assert names == [None, None, "k_fw_decode"] + ["k_fw_diag", "k_fw_panel", "k_fw_rest"] * tiles + [None]
        assert "k_weights" in got[1] and "k_fw_store" in got[-1]
    else:  # (2100: the integers in tiles of 128 and the value ranks in tiles of 64, each gated)
        assert names.count("k_fw_diag") == tiles
        assert names.count("k_fw_decode") == (m >= 1024)
