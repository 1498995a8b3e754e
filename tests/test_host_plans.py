"""What attention calls lay out in their workspace and launch, on contexts without a device: a C++ program in the place
of the kernels' launchers sees every descriptor (tests/host_sanitize/plans_host.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_20878_amd", "csrc")
HOST_SOURCES = ["ha_rag_api.hip", "ha_rag_pool.hip", "ha_rag_load.hip", "ha_rag_attend.hip", "ha_rag_io.hip"]
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")

OK, ENOSPC = 0, -3
SHARED2, SHARED4, ROLES4, ROLES8 = 20, 40, 41, 81  # forms of the shared kernel


@pytest.fixture(scope="module")
def plans_host(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plans") / "plans_host")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O1", "-g", "-std=c++17",
           "-Xarch_host", "-fsanitize=address,undefined", "-Xarch_host", "-fno-omit-frame-pointer",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
           "-x", "hip", os.path.join(ROOT, "tests", "host_sanitize", "plans_host.cpp"),
           *[os.path.join(CSRC, f) for f in HOST_SOURCES], "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def run(exe, args, text=None):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0", UBSAN_OPTIONS="halt_on_error=1")
    r = subprocess.run([exe, *args], input=text, capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    return r.stdout


def calls(exe, lines):
    """Per line: return code, workspace bytes, end of the last record, form, pieces, runs, longest run."""
    return [[int(x) for x in l.split()] for l in run(exe, ["calls"], "\n".join(lines) + "\n").splitlines()]


# Documents enough for a run to end because it may hold no more of them, next to ones long enough for runs to be long:
# the requests then have more runs than blocks / run length says.
MANY_DOCUMENTS = [
    "8 32" + " / 12 128*256 / 64 16*130" * 4,
    "16 64" + " / 32 1580*29 8*298" * 11,
    "8 64 / 16 944*106 / 256 16*176 / 16 96*134 / 16 / 16 / 16",
]


@pytest.mark.parametrize("how,codes", [("workspace", [OK, OK, OK]), ("static", [ENOSPC, ENOSPC, OK])])
def test_records_lie_in_the_workspace_when_runs_end_at_the_most_documents(plans_host, how, codes):
    seen = calls(plans_host, [how + " " + c for c in MANY_DOCUMENTS])
    assert [s[0] for s in seen] == codes
    for rc, need, end, *_ in seen:
        assert end <= (need if how == "workspace" else 32 << 20)


def test_random_calls_lay_every_record_out_once_and_inside(plans_host):
    assert "plans_host ok" in run(plans_host, ["random", "7", "2500"])


def test_planning_takes_less_than_the_descriptors_of_a_batch(plans_host):
    """Run lengths and forms are found without trying every length: long documents cost no more to plan than 320 short
    ones cost to list.  (Trying every one three or four times took 2.4, 11 and 49 times as long.)"""
    batch = "time 200 8 32" + " / 1 512*10" * 32
    rows = ["time 200 8 32 / 16 1024*16", "time 200 8 32 / 16 4096*32", "time 100 8 32 / 16 65536*32"]
    out = [l.split() for l in run(plans_host, ["calls"], "\n".join([batch] + rows) + "\n").splitlines()]
    assert all(rc == "0" for rc, _ in out)
    for _, us in out[1:]:
        assert float(us) < float(out[0][1]), out


# ---- the rule that workspaces are sized by, every run length tried -----------------------------------------


def longest_steps(lens, run, per_step):
    most, steps, left = 0, 0, run
    for n in lens:
        while n:
            take = min(n, left)
            steps += -(-take // per_step)
            n, left = n - take, left - take
            if not left:
                most, steps, left = max(most, steps), 0, run
    return max(most, steps)


def limit_words(H, reqs, tiles_waves, in_steps):
    """reqs: (tiles, blocks of each document).  Words with runs as long as costs least, each length tried."""
    if not reqs:
        return 0
    _, waves, side, per_block = tiles_waves
    largest = max((lens for _, lens in reqs), key=sum)
    per_step = waves if in_steps else 1
    blocks = sum(largest)
    all_steps = sum(-(-n // per_step) for n in largest)
    least = fewest = None
    best = chosen = blocks
    for n in range(1, blocks + 1):
        run = -(-blocks // n)
        if n > 1 and run < 8:
            break
        runs = [-(-sum(lens) // run) for _, lens in reqs]
        wgs = sum(k * H * -(-mt // (2 * waves)) for k, (mt, _) in zip(runs, reqs))
        recs = sum(k * H * mt for k, (mt, _) in zip(runs, reqs) if k > 1)
        rounds = -(-wgs // side)
        steps = max(-(-run // per_step), -(-all_steps // n))
        if len(largest) <= 32:
            steps = max(steps, longest_steps(largest, run, per_step))
        cost = rounds * (steps * per_step + 8) + recs // per_block
        if least is None or cost < least:
            least, best = cost, run
        if fewest is None or rounds * run < fewest:
            fewest, chosen = rounds * run, best
        if wgs >= 64 * side:
            break
    return sum(k * H * mt for k, mt in ((-(-sum(lens) // chosen), mt) for mt, lens in reqs) if k > 1) * 2080


def piece_words(H, reqs):
    def groups(piece):
        return sum(-(-n // piece) * H * -(-mt // 2) for mt, lens in reqs for n in lens)
    piece = 128
    while piece > 8 and groups(piece) < 2048:
        piece //= 2
    if piece == 8 and groups(4) <= 1024:
        piece = 4
    total = 0
    for mt, lens in reqs:
        for n in lens:
            parts = -(-n // piece)
            total += -(-n // -(-n // parts)) * H * mt
    return total * 2080


def test_workspace_sizes_are_those_of_the_rule(plans_host):
    import random
    rnd = random.Random(11)
    lines, expect = [], []
    for _ in range(300):
        H, G = rnd.choice([1, 2, 8, 16]), rnd.choice([1, 4, 8])
        most_q = rnd.choice([8, 16, 40, 200])
        same = rnd.random() < 0.3
        first = [max(1, int(2 ** rnd.uniform(0, 11))) for _ in range(rnd.randint(1, 12))]
        reqs, text = [], ""
        for _ in range(max(1, int(2 ** rnd.uniform(0, 5.3)))):
            lens = first if same else [max(1, int(2 ** rnd.uniform(0, 11))) for _ in range(rnd.randint(0, 12 if rnd.random() < 0.9 else 40))]
            n_q = rnd.randint(1, most_q)
            reqs.append((-(-n_q * G // 16), [-(-t // 16) for t in lens]))
            text += " / %d %s" % (n_q, " ".join(map(str, lens)))
        most = max(mt for mt, _ in reqs)
        rule = (4, 2, 1024, 600) if most <= 4 else (8, 4, 512, 450) if most <= 8 else (0, 8, 256, 280)
        some = [(mt, lens) for mt, lens in reqs if lens]

        def words(split):
            return piece_words(H, [r for r in some if r[0] <= split]) + limit_words(H, [r for r in some if r[0] > split], rule, True)
        total = words(2)
        if 2 < most <= 4:
            total = min(total, words(1))
        lines.append("workspace %d %d%s" % (H, H * G, text))
        expect.append(4 * total)
    assert [c[1] for c in calls(plans_host, lines)] == expect


@pytest.mark.parametrize("many,few,alone", [(31, 1, True), (28, 4, True), (16, 16, False), (15, 1, False), (7, 1, False), (1, 1, False)])
def test_two_tile_requests_join_ones_of_eight_tiles_where_one_launch_costs_less(plans_host, many, few, alone):
    """10 x 512 tokens, `few` requests of 32 query tokens (8 tiles) and `many` of 8 (2 tiles): most of a batch alone, a few
    with the others."""
    text = " / 32 512*10" * few + " / 8 512*10" * many
    (rc, need, end, taken, pieces, runs, _), = calls(plans_host, ["workspace 8 32" + text])
    assert rc == OK and end <= need and taken == ROLES4
    assert (pieces > 0) == alone


def call_line(n_reqs, n_docs, tokens, n_q, G, tag=2):
    """One call over 8 KV heads; document lengths and query tokens taken in turn."""
    text = "workspace 8 %d" % (8 * G)
    for r in range(n_reqs):
        text += " / %d" % n_q[r % len(n_q)]
        text += "".join(" %d*1*%d" % (tokens[(r * n_docs + i) % len(tokens)], tag) for i in range(n_docs))
    return text


def form(exe, *shape):
    """The form a call takes and its longest run."""
    (rc, need, end, taken, _, _, longest), = calls(exe, [call_line(*shape)])
    assert rc == OK and end <= need
    return taken, longest


@pytest.mark.parametrize("shape,taken", [
    ((10, 4, [256], [31], 8), ROLES8),     # 16 tiles: 32.8 us in two runs of eight scorers, 35.6 in one of four
    ((24, 2, [700, 333], [8, 7, 4], 8), SHARED2),  # up to four tiles: 30.2 us in k6_attend_shared, 33.8
    ((20, 1, [256], [5, 7, 7], 8), ROLES4)])    # 15.1 us, 18.8 in k6_attend_shared
def test_a_run_that_writes_the_output_itself_pays_for_its_end(plans_host, shape, taken):
    assert form(plans_host, *shape)[0] == taken


@pytest.mark.parametrize("shape,taken", [
    # 5 to 7 workgroups a head in 5 runs: 31 for the 32 places of an XCD, but 9 for the 8 of one engine
    ((5, 13, [100, 300], [163, 209, 142], 4), (ROLES8, 59)),   # 85.9 us, 146.8 with four scorers in one run
    # 2 to 4 workgroups a head in 9 runs: 30 for 32 places, 9 for 8
    ((6, 1, [700, 333], [47, 114, 105], 4), (ROLES8, 15)),     # 28.4 us, 37.0 with four scorers in runs of 22 blocks
    # as uneven, but every engine has a place for each
    ((7, 2, [700, 333], [40, 23, 106, 33], 8), (ROLES4, 65)),  # 36.3 us, 53.6 with eight scorers
    ((3, 4, [256], [179, 76, 69], 4), (ROLES8, 16))])          # 25.0 us, 33.3 with four scorers
def test_requests_of_different_widths_are_counted_by_engine(plans_host, shape, taken):
    assert form(plans_host, *shape) == taken


@pytest.mark.parametrize("shape,taken", [
    ((29, 2, [700, 333], [123, 160, 72], 4, 0), ROLES8),   # 113.9 us in three rounds, 140.8 in four of four scorers
    ((26, 3, [256], [20, 38, 21], 8), ROLES4)])            # 57.4 us, 64.6 in two rounds of eight
def test_later_rounds_of_eight_scorers_count_less(plans_host, shape, taken):
    assert form(plans_host, *shape)[0] == taken


@pytest.mark.parametrize("shape,taken", [
    ((12, 11, [129], [8, 13, 14], 8, 3), SHARED4),  # 33.1 us, 38.7 with four scorers
    ((18, 11, [1024], [10], 8, 3), SHARED4),        # 150 us, 177
    ((27, 2, [256], [18], 4, 1), ROLES4),           # 23.0 us, 26.1 in k6_attend_shared
    ((4, 12, [700, 333], [28], 4, 5), ROLES4)])  # 37.0 us, 40.1
def test_four_scorers_or_four_waves_that_do_both(plans_host, shape, taken):
    assert form(plans_host, *shape)[0] == taken


def test_steps_of_few_blocks_count_less_for_eight_scorers_too(plans_host):
    assert form(plans_host, 5, 7, [304, 144, 600], [96], 4)[0] == ROLES8     # 45.3 us, 49.7 with four scorers
    assert form(plans_host, 19, 1, [100, 300], [55, 246, 148], 4, 0)[0] == ROLES8  # 46.7 us, 56.9


def requests_line(H, G, reqs):
    """reqs as tests/test_gpu_attend.py lists them."""
    return "workspace %d %d" % (H, H * G) + "".join(
        " / %d" % n_q + "".join(" %d*1*%d" % tp for tp in zip(tokens, precs)) for tokens, precs, n_q in reqs)


def test_gpu_tests_of_the_forms_take_the_forms_that_they_name(plans_host):
    import test_gpu_attend as gpu
    lines = [requests_line(1, 4, gpu.form_call(n_q, *call)) for call in gpu.FORM_CALLS for n_q in gpu.FORM_QUERIES]
    lines += [requests_line(1, 4, gpu.batch_call(n_q)) for n_q in gpu.FORM_QUERIES]
    assert [c[3] for c in calls(plans_host, lines)] == \
        [ROLES4] * 21 + [SHARED2, SHARED2, SHARED4, SHARED4, ROLES8, ROLES8, ROLES8]
    for n_q, H in ((9, 256), (33, 64)):
        (rc, need, end, _, _, runs, longest), = calls(plans_host, [requests_line(H, 4, gpu.long_lists_call(n_q))])
        assert rc == OK and end == need and (runs, longest) == (8, 128)


# ---- loads past the last-level cache ------------------------------------------------------------------------
BF16, INT8, INT4, E4M3, GSE8 = 0, 1, 2, 3, 5
MIX = [BF16] * 2 + [INT8] * 3 + [INT4] * 5  # 20 / 30 / 50 %: 10.2 MB a layer for ten documents of 512 tokens


def past_line(layers, n_reqs, n_docs, tokens, tags, H=8, n_q=1, apart=1 << 24, back=0):
    """back: the documents of the last `back[0]` requests are those of `back[1]` requests before."""
    text = "past %d %d %d %d" % (layers, apart, H, 4 * H)
    for r in range(n_reqs):
        again = back[1] * n_docs if back and r >= n_reqs - back[0] else 0
        text += " / %d" % n_q + "".join(" %d*1*%d*%d" % (tokens, tags[i % len(tags)], again) for i in range(n_docs))
    return text


def reads_past(exe, *shape, **more):
    (rc, past, _), = calls(exe, [past_line(*shape, **more)])
    assert rc == OK
    return bool(past)


@pytest.mark.parametrize("shape,past", [
    # us a pass, ordinary / nontemporal loads
    ((2, 32, 10, 512, MIX), True),         # 655 MB: 151 / 141
    ((2, 27, 10, 512, MIX), True),         # 551 MB: 130 / 122
    ((2, 23, 10, 512, MIX), False),        # 465 MB, 16 blocks: 115 / 116
    ((1, 29, 10, 512, MIX), False),        # 297 MB in one layer: 60 / 64 at 302
    ((4, 12, 10, 512, MIX), False),        # 491 MB, eight blocks, 3,840 workgroups: 142 / 154 at 467 MB
    ((1, 20, 10, 512, [BF16]), False),     # 419 MB, 16 blocks: 83 / 89
    ((2, 10, 10, 512, [BF16]), False),     # 419 MB, eight blocks: 101 / 118
    ((1, 30, 10, 512, [BF16]), True),      # 629 MB, 32 blocks: 118 / 114
    ((2, 16, 10, 512, [E4M3]), True),      # 336 MB: 80 / 77
    ((2, 15, 10, 512, [E4M3]), False),     # 315 MB
    ((8, 5, 9, 512, [GSE8]), True),        # 377 MB, pieces of eight blocks: 166 / 159
    ((32, 1, 10, 512, MIX), False),        # one request, 327 MB: 369 / 358, with the cache full of other data 14.5 / 14.8 a layer
    ((32, 2, 10, 512, MIX), True),         # two, 655 MB, eight blocks, 640 workgroups: 439 / 421
    ((32, 6, 10, 512, MIX), False),        # 1,920 workgroups: 763 / 768
    ((32, 2, 10, 512, [BF16]), False),     # 492 / 501
    ((32, 2, 10, 512, [INT8]), True)])     # 694 MB
def test_documents_are_read_past_the_cache_where_that_is_faster(plans_host, shape, past):
    assert reads_past(plans_host, *shape) == past


def test_gpu_tests_of_loads_past_the_cache_take_the_builds_that_they_name(plans_host):
    import test_gpu_attend as gpu
    for with_16_bit, many, H, reqs in gpu.PAST_CALLS:
        text = "".join(" / 1" + "".join(" %d*1*%d*0*1 %d*1*%d*0*2" % (t, k, t, v) for t, k, v in docs) for docs in reqs)
        (rc, past, pieces), (rc1, past1, _) = calls(plans_host, ["past %d %d %d %d" % (n, 1 << 24, H, H) + text for n in (gpu.PAST_LAYERS, 1)])
        assert rc == rc1 == OK and past and not past1
        assert (pieces > 8192 // 72) == many  # the structure of few holds 113 runs


def test_documents_in_pinned_host_memory_are_read_with_ordinary_loads(plans_host):
    """In the pool's slab by id and by address, at addresses of the caller's by id; none of them there first."""
    assert run(plans_host, ["pinned", "1"]).split() == ["1", "1", "1", "0", "0", "0"]


@pytest.mark.parametrize("shape,apart", [((2, 32, 10, 657, [BF16]), 5505024), ((1, 32, 32, 433, [BF16]), 1835008), ((2, 64, 32, 128, [E4M3]), 1 << 20),
                                         ((2, 64, 64, 64, [E4M3]), 4096)])
def test_documents_at_even_distances_are_not_taken_for_repeated_ones(plans_host, shape, apart):
    assert reads_past(plans_host, *shape, apart=apart)


@pytest.mark.parametrize("shape,back,past", [
    ((2, 32, 10, 512, [E4M3]), (8, 8), True),      # a quarter listed before: 114 us with ordinary loads, 109 with nontemporal ones
    ((2, 32, 10, 512, [E4M3]), (8, 24), True),     # after all others: 128 / 123
    ((2, 32, 10, 512, [E4M3]), (16, 16), False),   # half: 115 / 121
    ((2, 32, 10, 512, MIX), (4, 4), True),         # an eighth
    ((2, 32, 10, 512, MIX), (8, 24), False),       # a quarter: 133 / 138
    ((2, 18, 10, 512, [E4M3]), (4, 14), False),    # 377 MB listed, 293 MB of documents
    ((2, 64, 32, 128, [E4M3]), (32, 32), False),   # 2,048 documents, the second half as the first
    ((1, 128, 32, 128, [E4M3]), (16, 112), True)]) # 4,096, an eighth listed before
def test_repeated_documents_count_once(plans_host, shape, back, past):
    assert reads_past(plans_host, *shape, back=back) == past


# ---- tiles of short GSE-8 chunks that share workgroups -------------------------------------------------------


@pytest.mark.parametrize("n_tiles,tokens,per_wg", [
    (32, [30] * 40 + [1024], [1] * 41),                     # 24 us; 16 in one, on two XCDs, 46
    (32, [300] * 20 + [40] * 20, [1] * 40),                 # 19 / 25
    (512, [600, 40], [1, 2]),                               # 28.0 alone, 26.6, 32.3 with 16 in one
    (256, [16, 44, 64, 1024], [3, 3, 3, 1]),                # 25.8 alone, 23.5, 29.2 with 16
    (512, [1024, 300, 300, 300], [1] * 4),                  # 75.7, 81 with three
    (512, [16, 16, 16, 16, 512], [16] * 4 + [1]),           # 29.8 alone, 24.7
    (128, [16] * 12 + [1024], [4] * 12 + [1]),              # 27 alone, 19.8
    (128, [33, 17, 60, 512], [1] * 4),                      # as many as there are places
    (512, [64, 20], [1, 1]),                                # workgroups of four waves, eight to a compute unit
    (512, [64, 20] * 3, [1, 2] * 3),
    (512, [2000] + [100] * 6, [1] * 7)])                    # tiles that are read twice
def test_tiles_share_workgroups_where_that_is_faster(plans_host, n_tiles, tokens, per_wg):
    assert [int(x) for x in run(plans_host, ["share", str(n_tiles), *map(str, tokens)]).split()] == per_wg


def test_shared_workgroups_have_the_waves_that_their_tiles_need(plans_host):
    import random
    rnd = random.Random(3)
    for _ in range(60):
        tokens = [max(1, int(2 ** rnd.uniform(0, rnd.choice([4, 8, 10, 11])))) for _ in range(rnd.randint(1, 128))]
        run(plans_host, ["share", str(rnd.choice([2, 8, 33, 64, 264, 1280])), *map(str, tokens)])


@pytest.mark.parametrize("n_q", [12, 80])
def test_gpu_tests_at_the_edge_of_few_descriptors_end_where_they_say(plans_host, n_q):
    import test_gpu_attend as gpu
    lines = ["ends 1 8 / %d" % n_q + "".join(" %d*1*%d" % (t, (INT4, BF16, GSE8)[i % 3]) for i, t in enumerate(tokens))
             for tokens in gpu.EDGE_DOCUMENTS.values()]
    assert calls(plans_host, lines) == [[OK, end] for end in gpu.EDGE_DOCUMENTS]
