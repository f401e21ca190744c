"""The C ABI on the CPU: the library loads, exports every declared symbol,
validates arguments before launching anything, and its host-side role
allocation agrees with the oracle."""

import ctypes
import os
import re

import numpy as np
import pytest

import oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def kve():
    from paper_2607_13205_amd.build import ensure_built
    ensure_built()
    import paper_2607_13205_amd as K
    return K


def _declared():
    text = open(os.path.join(ROOT, "include", "kve.h")).read()
    return sorted(set(re.findall(r"\b(kve_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(kve):
    names = _declared()
    assert len(names) == 29
    assert sorted(kve.EXPORTED) == names
    lib = ctypes.CDLL(kve.binding._LIB_PATH)
    for n in names:
        assert hasattr(lib, n), n
    assert kve.binding.LIB.kve_version() == 1


def test_library_reports_the_hash_of_its_sources(kve):
    """The loaded library was built from the present csrc/ and include/ (the
    build embeds the hash; ensure_built rebuilds when the sources change)."""
    from paper_2607_13205_amd.build import built_hash, source_hash
    h = kve.source_hash()
    assert re.fullmatch(r"[0-9a-f]{64}", h), h
    assert h == source_hash() == built_hash()


@pytest.mark.parametrize("ex_seed", range(3))
def test_role_allocate_matches_oracle_on_random_grid(kve, ex_seed):
    r = np.random.default_rng(ex_seed)
    for _ in range(400):
        N = int(r.integers(1, 300))
        W = int(r.integers(0, N + 1))
        R = int(r.integers(1, 9))
        B = int(r.integers(1, 4))
        roles = r.integers(0, R, (B, N)).astype(np.int8)
        alpha = r.random(R)
        alpha[r.random(R) < 0.3] = 0.0
        if alpha.sum() == 0:
            alpha[-1] = 0.5
        budget = float(r.choice([0.01, 0.05, 0.07, 0.1, 0.2, 0.33, 0.5, 0.9, 1.0, 1.5]))
        q, kept, kcap = kve.role_allocate(roles, R, alpha, budget, W)
        qo, ko, kco = O.role_allocate_batch(roles, R, alpha, budget, W)
        assert np.array_equal(q, qo) and np.array_equal(kept, ko) and kcap == kco


def test_role_allocate_golden_examples(kve):
    from tests.test_oracle_alloc import _load_examples, _roles_from_counts
    for name, N, W, B, alpha, n, quota, kept in _load_examples():
        roles = _roles_from_counts(n, W)
        q, k, _ = kve.role_allocate(roles, 4, alpha, B, W)
        assert q[0].tolist() == quota and int(k[0]) == kept, name


def test_role_allocate_rejects_bad_input(kve):
    roles = np.zeros((1, 10), dtype=np.int8)
    a = [0.25, 0.0, 0.7, 0.05]
    for args in [(roles, 4, a, 0.0, 2), (roles, 4, a, 0.5, 11), (roles, 9, a * 3, 0.5, 2),
                 (roles, 4, [0, 0, 0, 0], 0.5, 2), (roles, 4, [0.1, -1, 0.7, 0.05], 0.5, 2),
                 (roles + 4, 4, a, 0.5, 2), (roles, 4, a, float("nan"), 2)]:
        with pytest.raises(kve.KveError) as e:
            kve.role_allocate(*args)
        assert e.value.status == 1
        assert kve.last_error()


@pytest.mark.parametrize("ex_seed", range(3))
def test_fair_allocate_matches_oracle_on_random_grid(kve, ex_seed):
    r = np.random.default_rng(50 + ex_seed)
    for _ in range(400):
        N = int(r.integers(1, 300))
        W = int(r.integers(0, N + 1))
        R = int(r.integers(1, 9))
        B = int(r.integers(1, 4))
        p = r.dirichlet(np.full(R, 0.5))
        roles = r.choice(R, (B, N), p=p).astype(np.int8)
        budget = float(r.choice([0.01, 0.05, 0.07, 0.1, 0.2, 0.33, 0.5, 0.9, 1.0, 1.5]))
        q, kept, kcap = kve.role_allocate_fair(roles, R, budget, W)
        qo, ko, kco = O.fair_allocate_batch(roles, R, budget, W)
        assert np.array_equal(q, qo) and np.array_equal(kept, ko) and kcap == kco


def test_role_map_and_no_role_allocation_match_oracle(kve):
    r = np.random.default_rng(60)
    for _ in range(200):
        n_roles = int(r.integers(2, 6))
        B, N = int(r.integers(1, 4)), int(r.integers(1, 300))
        W = int(r.integers(0, N + 1))
        roles = r.integers(0, n_roles, (B, N)).astype(np.int8)
        x = int(r.integers(0, n_roles))
        bucket_of, alpha = O.no_role_policy(x, n_roles)
        buckets = kve.role_map(roles, bucket_of)
        assert np.array_equal(buckets, O.role_map(roles, bucket_of))
        budget = float(r.choice([0.05, 0.1, 0.3, 0.5, 1.0]))
        q, kept, kcap = kve.role_allocate(buckets, 2, alpha, budget, W)
        qo, ko, kco = O.role_allocate_batch(O.role_map(roles, bucket_of), 2, alpha, budget, W)
        assert np.array_equal(q, qo) and np.array_equal(kept, ko) and kcap == kco
    # an arbitrary many-to-one map
    roles = r.integers(0, 7, (2, 100)).astype(np.int8)
    bmap = [3, 0, 7, 7, 1, 0, 2]
    assert np.array_equal(kve.role_map(roles, bmap), O.role_map(roles, bmap))


def test_fair_and_map_reject_bad_input(kve):
    roles = np.zeros((1, 10), dtype=np.int8)
    for args in [(roles, 4, 0.0, 2), (roles, 4, 0.5, 11), (roles, 9, 0.5, 2), (roles + 4, 4, 0.5, 2),
                 (roles, 4, float("inf"), 2)]:
        with pytest.raises(kve.KveError) as e:
            kve.role_allocate_fair(*args)
        assert e.value.status == 1
    for rl, bmap in [(roles + 3, [0, 1, 0]), (roles, [8, 0]), (roles, [-1]),
                     (roles, [0] * 128)]:
        out_before = rl.copy()
        with pytest.raises(kve.KveError) as e:
            kve.role_map(rl, bmap)
        assert e.value.status == 1 and np.array_equal(rl, out_before)


def test_device_entry_points_validate_before_launch(kve):
    """Invalid arguments return an error code without touching the GPU (no
    device exists here, so any launch would fail with KVE_ERR_HIP instead)."""
    L = kve.binding.LIB
    null = None
    dummy = ctypes.c_void_p(0x1000)  # never dereferenced: every call below fails validation
    # snapkv: even pool kernel, W > N, unsupported d, Hq % Hkv, short workspace, null score
    assert L.kve_snapkv_score(dummy, dummy, 0, 1, 1, 4, 2, 64, 8, 128, 0.0, 4, dummy, dummy, 1 << 30, null) == 1
    assert L.kve_snapkv_score(dummy, dummy, 0, 1, 1, 4, 2, 64, 65, 128, 0.0, 7, dummy, dummy, 1 << 30, null) == 1
    assert L.kve_snapkv_score(dummy, dummy, 0, 1, 1, 4, 2, 64, 8, 96, 0.0, 7, dummy, dummy, 1 << 30, null) == 2
    assert L.kve_snapkv_score(dummy, dummy, 0, 1, 1, 5, 2, 64, 8, 128, 0.0, 7, dummy, dummy, 1 << 30, null) == 1
    assert L.kve_snapkv_score(dummy, dummy, 0, 1, 1, 4, 2, 64, 8, 128, 0.0, 7, dummy, dummy, 16, null) == 3
    assert L.kve_snapkv_score(dummy, dummy, 0, 1, 1, 4, 2, 64, 8, 128, 0.0, 7, null, dummy, 1 << 30, null) == 1
    assert L.kve_snapkv_score(dummy, dummy, 7, 1, 1, 4, 2, 64, 8, 128, 0.0, 7, dummy, dummy, 1 << 30, null) == 2
    assert L.kve_snapkv_score(dummy, dummy, 0, 1, 1, 64, 1, 64, 32, 128, 0.0, 7, dummy, dummy, 1 << 30, null) == 2
    assert "pool_k" in kve.last_error() or kve.last_error()
    # snapkv with supplied row statistics: null lse_win, and the same checks as the plain score
    assert L.kve_snapkv_score_lse(dummy, dummy, null, 0, 1, 1, 4, 2, 64, 8, 128, 0.0, 7, dummy, dummy, 1 << 30, null) == 1
    assert L.kve_snapkv_score_lse(dummy, dummy, dummy, 0, 1, 1, 4, 2, 64, 8, 128, 0.0, 4, dummy, dummy, 1 << 30, null) == 1
    assert L.kve_snapkv_score_lse(dummy, dummy, dummy, 0, 1, 1, 4, 2, 64, 8, 128, 0.0, 7, dummy, dummy, 16, null) == 3
    # h2o: short workspace, bad dtype
    assert L.kve_h2o_score(dummy, dummy, 0, 1, 1, 4, 2, 64, 128, 0.0, dummy, dummy, 8, null) == 3
    assert L.kve_h2o_score(dummy, dummy, 3, 1, 1, 4, 2, 64, 128, 0.0, dummy, dummy, 1 << 30, null) == 2
    # topk: R out of range, W > N, negative k_cap
    assert L.kve_topk_select(dummy, dummy, dummy, 1, 1, 2, 64, 8, 9, 10, dummy, dummy, null, 0, null) == 1
    assert L.kve_topk_select(dummy, dummy, dummy, 1, 1, 2, 64, 65, 4, 10, dummy, dummy, null, 0, null) == 1
    assert L.kve_topk_select(dummy, dummy, dummy, 1, 1, 2, 64, 8, 4, -1, dummy, dummy, null, 0, null) == 1
    # topk: no workspace, a short one, a misaligned one
    assert L.kve_topk_select(dummy, dummy, dummy, 1, 1, 2, 64, 8, 4, 10, dummy, dummy, null, 0, null) == 3
    assert L.kve_topk_select(dummy, dummy, dummy, 1, 1, 2, 64, 8, 4, 10, dummy, dummy, dummy, 1023, null) == 3
    assert L.kve_topk_select(dummy, dummy, dummy, 1, 1, 2, 64, 8, 4, 10, dummy, dummy,
                             ctypes.c_void_p(0x1008), 1 << 20, null) == 1
    # compact: v without v_out, bad head_dim
    assert L.kve_kv_compact(dummy, dummy, 0, dummy, dummy, 1, 1, 2, 64, 128, 10, dummy, null, null) == 1
    assert L.kve_kv_compact(dummy, null, 0, dummy, dummy, 1, 1, 2, 64, 80, 10, dummy, null, null) == 2
    big = 1 << 30
    # probe: R out of range, null ids, empty batch
    assert L.kve_role_probe(dummy, 1, 10, dummy, dummy, 100, 9, dummy, null) == 1
    assert L.kve_role_probe(null, 1, 10, dummy, dummy, 100, 6, dummy, null) == 1
    assert L.kve_role_probe(dummy, 0, 10, dummy, dummy, 100, 6, dummy, null) == 1
    # quest: page 0, page too large, W > N, G > 8, short workspace
    assert L.kve_quest_score(dummy, dummy, 0, 1, 1, 8, 2, 64, 8, 128, 0, dummy, dummy, big, null) == 1
    assert L.kve_quest_score(dummy, dummy, 0, 1, 1, 8, 2, 64, 8, 128, 2000, dummy, dummy, big, null) == 1
    assert L.kve_quest_score(dummy, dummy, 0, 1, 1, 8, 2, 64, 65, 128, 16, dummy, dummy, big, null) == 1
    assert L.kve_quest_score(dummy, dummy, 0, 1, 1, 18, 2, 64, 8, 128, 16, dummy, dummy, big, null) == 2
    assert L.kve_quest_score(dummy, dummy, 0, 1, 1, 8, 2, 64, 8, 128, 16, dummy, dummy, 8, null) == 3
    # decode: G > 8, null count, short workspace, negative scale, k_cap 0, misaligned workspace
    assert L.kve_decode_attention(dummy, dummy, dummy, dummy, 0, 1, 1, 18, 2, 64, 128, 0.0, dummy, dummy, big, null) == 2
    assert L.kve_decode_attention(dummy, dummy, dummy, null, 0, 1, 1, 8, 2, 64, 128, 0.0, dummy, dummy, big, null) == 1
    assert L.kve_decode_attention(dummy, dummy, dummy, dummy, 0, 1, 1, 8, 2, 64, 128, 0.0, dummy, dummy, 8, null) == 3
    assert L.kve_decode_attention(dummy, dummy, dummy, dummy, 0, 1, 1, 8, 2, 64, 128, -1.0, dummy, dummy, big, null) == 1
    assert L.kve_decode_attention(dummy, dummy, dummy, dummy, 0, 1, 1, 8, 2, 0, 128, 0.0, dummy, dummy, big, null) == 1
    assert L.kve_decode_attention(dummy, dummy, dummy, dummy, 0, 1, 1, 8, 2, 64, 128, 0.0, dummy,
                                  ctypes.c_void_p(0x1010), big, null) == 1


def test_workspace_sizes_are_aligned_and_monotone(kve):
    a = kve.snapkv_workspace_size(1, 1, 32, 8, 8192, 32, 128)
    b = kve.snapkv_workspace_size(2, 1, 32, 8, 8192, 32, 128)
    assert a > 0 and a % 256 == 0 and b >= a
    # one start value per query row (rows padded to 64 floats) and one column sum
    # per (query head, key)
    assert kve.h2o_workspace_size(1, 1, 32, 8, 16384, 128) == 2 * 32 * 16384 * 4
    h = kve.h2o_workspace_size(2, 1, 32, 8, 1000, 128)
    assert h % 256 == 0 and h >= 2 * 32 * 1024 * 4 + 2 * 32 * 1000 * 4
    # top-k: one staged 8-byte entry per position of every segment
    assert kve.topk_workspace_size(1, 1, 8, 8192, 4) == 8 * 8192 * 8
    assert kve.topk_workspace_size(2, 3, 1, 1001, 4) == (6 * 1001 * 8 + 255) // 256 * 256
    assert kve.topk_workspace_size(1, 1, 8, 0, 4) == 0
    # decode: per (segment, split, head) a partial output row and a pair of floats
    w = kve.decode_workspace_size(32, 4, 32, 8, 1640, 128)
    assert w % 256 == 0 and w >= 1024 * 32 * (128 + 2) * 4 // 8
    assert kve.decode_workspace_size(1, 1, 32, 8, 0, 128) == 0
    assert kve.quest_workspace_size(2, 1, 32, 8, 128) == 2 * 32 * 128 * 4


def test_strided_entry_points_reject_bad_views_before_any_launch(kve):
    """View checks run on the host before anything touches the device (the
    pointers below are never dereferenced)."""
    lib = kve.binding.LIB
    S = kve.Strides
    fake = ctypes.c_void_p(0x10000)
    score = ctypes.c_void_p(0x20000)
    ws = ctypes.c_void_p(0x40000)
    dense_k = S(2 * 8 * 1024 * 128, 8 * 1024 * 128, 1024 * 128, 128)

    def score_call(qs, ks, q=fake):
        return lib.kve_snapkv_score_strided(q, None if qs is None else ctypes.byref(qs), fake,
                                            None if ks is None else ctypes.byref(ks), 0, 1, 2, 8, 8, 1024, 16,
                                            128, 0.0, 7, score, ws, 1 << 30, None)

    bad = [S(-128, 0, 0, 128),                      # negative stride
           S(0, 0, 0, 4),                           # 8 bytes: not a multiple of 16
           S(0, 0, 0, (1 << 24) + 8)]               # token stride above 2^25 bytes
    for st in bad:
        assert score_call(None, st) == kve.binding.KVE_ERR_INVALID_ARG, st
        assert "stride" in kve.last_error()
        assert score_call(st, dense_k) == kve.binding.KVE_ERR_INVALID_ARG
    # a misaligned base pointer of a strided view
    assert score_call(S(0, 0, 16 * 128, 128), None, q=ctypes.c_void_p(0x10008)) == kve.binding.KVE_ERR_INVALID_ARG
    assert "aligned" in kve.last_error()
    idx = ctypes.c_void_p(0x50000)
    cnt = ctypes.c_void_p(0x60000)
    out = ctypes.c_void_p(0x70000)
    st = lib.kve_kv_compact_strided(fake, ctypes.byref(dense_k), fake, ctypes.byref(S(0, 0, -1, 128)), 0, idx,
                                    cnt, 1, 2, 8, 1024, 128, 64, out, out, None)
    assert st == kve.binding.KVE_ERR_INVALID_ARG and "negative" in kve.last_error()


def test_snapkv_rejects_more_window_rows_than_supported_before_any_launch(kve):
    """G*W above 1024 window rows per KV head is refused on the host (the
    pointers are never dereferenced); 1024 itself passes the check and fails
    only later, on the fake workspace size."""
    lib = kve.binding.LIB
    fake = ctypes.c_void_p(0x10000)
    score = ctypes.c_void_p(0x20000)
    ws = ctypes.c_void_p(0x40000)
    # Hq = 16, Hkv = 1, W = 65: 1040 rows
    st = lib.kve_snapkv_score(fake, fake, 0, 1, 1, 16, 1, 4096, 65, 128, 0.0, 7, score, ws, 1 << 30, None)
    assert st == kve.binding.KVE_ERR_UNSUPPORTED and "1024" in kve.last_error()
    # W = 64: 1024 rows, accepted by the row check, refused for the 16-byte workspace
    st = lib.kve_snapkv_score(fake, fake, 0, 1, 1, 16, 1, 4096, 64, 128, 0.0, 7, score, ws, 16, None)
    assert st == kve.binding.KVE_ERR_WORKSPACE


def _run_plan(tmp_path, program, args):
    """Lines that a program over one of the plain C++ plan headers prints."""
    import os
    import shutil
    import subprocess
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "plan.cpp", str(tmp_path / "plan")
    src.write_text(program)
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_13205_amd", "csrc")
    subprocess.run([cxx, "-std=c++17", "-I", csrc, str(src), "-o", exe], check=True)
    out = subprocess.run([exe] + [str(x) for a in args for x in a], check=True, capture_output=True, text=True).stdout
    return out.strip().split("\n")


TOPK_PLAN_PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "kve_topk_plan.h"
int main(int argc, char** argv) {
    for (int i = 1; i + 2 < argc; i += 3) {
        const int segs = atoi(argv[i]), N = atoi(argv[i + 1]), R = atoi(argv[i + 2]);
        printf("%d %d\\n", (int)kve::topk_in_regs(segs, N, R), kve::topk_slices(segs, N, R));
    }
}
"""


def test_topk_slices_fit_the_chip_and_their_records(tmp_path):
    """Slices of split segments: one workgroup per compute unit for all of them
    (two per segment at least) unless 16-bit offsets need more, each with room
    for its counts (8 bytes per position: tags, offsets and 16-bit counts)."""
    cases = [(s, n, r) for s in (1, 2, 7, 8, 16, 33, 64, 65, 256, 1023, 1024) for r in (1, 2, 4, 5, 8)
             for n in (4096, 8192, 8193, 16384, 16385, 24000, 40001, 65536, 131071, 262144, 270001, 1000000, 4192256, 4192257)]
    for (segs, n, r), line in zip(cases, _run_plan(tmp_path, TOPK_PLAN_PROGRAM, cases)):
        regs, s = (int(x) for x in line.split())
        assert regs == (n <= (8192 if segs >= 1024 and r <= 4 else 16384)), (segs, n, r)
        if s == 0:
            assert segs > 64 or n > 64 * 65504 or n < 2 * max(4096, 2048 * r + 128), (segs, n, r)
            continue
        assert 2 <= s <= 64 and segs <= 64
        shortest, longest = n // 16 // s * 16, n // 16 // s * 16 + 32
        assert longest <= 65536, (segs, n, r, s)
        assert 2 * shortest >= 2 * 2048 * r + 16 + 112, (segs, n, r, s)
        assert s * segs <= max(256, 2 * segs) or s == -(-n // 65504), (segs, n, r, s)


SNAP_PLAN_PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "kve_snap_plan.h"
int main(int argc, char** argv) {
    for (int i = 1; i + 7 < argc; i += 8) {
        int a[8];
        for (int j = 0; j < 8; ++j) a[j] = atoi(argv[i + j]);
        const kve::SnapPlan p = kve::snap_plan(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7]);
        printf("%d %d %d\\n", p.n_vsegs * p.nranges, p.range_keys / 64, p.nranges);
    }
}
"""


def test_snapkv_ranges_fill_whole_groups_of_workgroups(tmp_path):
    """Where a score's key ranges make more workgroups than run together (four per
    compute unit, 16-bit rows in one set), their number is close to a multiple of
    that; 64-element rows take four per unit rather than fewer, longer ones; a
    short prompt keeps one or two per unit."""
    cases = [(8, 2, 8, 8, 81344, 64, 128, 2), (16, 2, 8, 8, 40000, 32, 128, 2), (8, 2, 8, 8, 81344, 32, 64, 2),
             (8, 1, 8, 8, 65536, 32, 64, 2), (4, 4, 8, 8, 14976, 16, 64, 2), (1, 1, 32, 8, 32768, 32, 128, 2),
             (1, 1, 32, 8, 8192, 32, 128, 2)]
    for case, line in zip(cases, _run_plan(tmp_path, SNAP_PLAN_PROGRAM, cases)):
        groups, per, ranges = (int(x) for x in line.split())
        assert per * ranges >= -(-case[4] // 64) > per * (ranges - 1), (case, line)
        rounds = -(-groups // 256)
        if case[4] > 10000 and (case[0] > 1 or case[6] == 64):
            assert rounds % 4 == 0, (case, line)
        else:
            assert rounds <= 2, (case, line)


QUEST_PLAN_PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "kve_quest_plan.h"
int main(int argc, char** argv) {
    for (int i = 1; i + 8 < argc; i += 9) {
        int a[9];
        for (int j = 0; j < 9; ++j) a[j] = atoi(argv[i + j]);
        const kve::QuestPlan p = kve::quest_plan(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8]);
        printf("%d %d %d\\n", p.n_pages, p.range_pages, p.nranges);
    }
}
"""


def test_quest_ranges_weigh_a_workgroups_start(tmp_path):
    """Ranges cover the pages; four steps of 16-key pages per workgroup with four
    heads and more per group, two where a start weighs less (float32, fewer
    heads), one of long pages until 4096 workgroups are full, and at most 32 of
    short ones."""
    #        L, B, Hq, Hkv, N, W, d, bytes, page, steps per workgroup
    cases = [(1, 1, 32, 8, 131072, 32, 128, 2, 16, 4), (4, 2, 32, 8, 24571, 32, 128, 2, 16, 4),
             (1, 3, 12, 3, 105344, 32, 128, 4, 16, 2), (4, 2, 8, 8, 28834, 64, 128, 2, 16, 2),
             (4, 1, 32, 8, 32768, 32, 128, 2, 1, 32), (8, 4, 8, 8, 5345, 32, 64, 4, 1, 16),
             (4, 3, 12, 3, 81792, 16, 128, 2, 64, 1), (8, 1, 32, 8, 32768, 32, 128, 4, 64, 4),
             (1, 1, 32, 8, 8192, 32, 128, 2, 16, 1)]
    for case, line in zip(cases, _run_plan(tmp_path, QUEST_PLAN_PROGRAM, [c[:9] for c in cases])):
        pages, per, ranges = (int(x) for x in line.split())
        assert per * ranges >= pages > per * (ranges - 1), (case, line)
        assert per == case[9] * 4 * (64 // (case[6] * case[7] // 16)), (case, line)


DECODE_PLAN_PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "kve_decode_plan.h"
int main(int argc, char** argv) {
    for (int i = 1; i + 2 < argc; i += 3) {
        const kve::DecodePlan p = kve::decode_plan(1, atoi(argv[i]), 4, 1, atoi(argv[i + 1]), atoi(argv[i + 2]));
        printf("%d %d %zu\\n", p.nsplit, p.split_keys / kve::kDecodeQuantum, p.off_ml);
    }
}
"""


def test_decode_splits_fill_the_compute_units(tmp_path):
    """Splits cover the cache and fit the workspace.  Short ones stay one
    workgroup per compute unit; of the others, unless they are already as short
    as three workgroups per unit make them, none is longer than 16 quanta (the
    counts of a batch differ) and the rounds of one workgroup per unit are at
    least 0.85 full."""
    cases = [(s, k, d) for s in (1, 2, 7, 8, 31, 32, 64, 96, 100, 128, 136, 160, 200, 248, 255, 256, 257, 264, 288, 320,
                                 384, 448, 504, 512, 513, 640, 800, 1016, 1023, 1024, 1025, 5000)
             for k in (1, 127, 128, 129, 400, 820, 1639, 2048, 2049, 3277, 6000, 20000, 32768, 200001)
             for d in (64, 128)]
    for (segs, k_cap, d), line in zip(cases, _run_plan(tmp_path, DECODE_PLAN_PROGRAM, cases)):
        ns, per, room = (int(x) for x in line.split())
        quanta = -(-k_cap // 128)
        assert ns * per >= quanta > (ns - 1) * per, (segs, k_cap, d, line)
        assert segs * ns * 4 * d * 4 <= room, (segs, k_cap, d, line)
        one = -(-quanta // min(quanta, -(-256 // segs)))  # quanta per split at one workgroup per unit
        whole = one >= quanta
        if one <= (7 if whole else 4) * (128 // d):
            assert per == one, (segs, k_cap, d, line)
            continue
        rounds = -(-segs * ns // 256)
        even = rounds == 1 or segs * ns >= 0.85 * 256 * rounds
        longest = 16 * (128 // d) if ns == 1 else 16
        least_of_three = -(-quanta // min(quanta, -(-768 // segs)))  # at three workgroups per unit
        assert (per <= longest and even) or per <= least_of_three, (segs, k_cap, d, line)


@pytest.mark.parametrize("L,B,Hq,Hkv,N,W,d", [(1, 1, 2, 1, 512, 16, 64), (1, 1, 32, 8, 8192, 32, 128),
                                              (8, 2, 32, 8, 20011, 32, 128), (1, 1, 32, 8, 131072, 64, 128),
                                              (32, 4, 32, 8, 32768, 32, 128), (2, 3, 12, 3, 5003, 50, 64)])
def test_workspace_sizes_do_not_follow_the_launch_rules(kve, L, B, Hq, Hkv, N, W, d):
    """The sizes are those of the smallest key ranges (score) and of 1024
    workgroups (decode), whatever a call's own plan takes."""
    def up(x):
        return (x + 255) // 256 * 256
    segs, rows, chunks = L * B * Hkv, Hq // Hkv * W, -(-N // 64)

    def score(elem):
        rpg = 256 if elem == 2 and rows > 128 else 128
        groups = -(-rows // rpg)
        per = -(-chunks * segs * groups // 4096)
        per = min(max(per, -(-min(rows, rpg) // 64)), 128, chunks)
        ranges = -(-chunks // per)
        return up(4 * segs * groups * ranges * rpg) + up(4 * segs * groups * rpg) + up(4 * groups * segs * N)
    assert kve.snapkv_workspace_size(L, B, Hq, Hkv, N, W, d) == max(score(2), score(4))
    assert kve.topk_workspace_size(L, B, Hkv, N, 4) == up(8 * segs * N)
    quanta = -(-N // 128)
    per = -(-quanta // max(1, min(quanta, -(-1024 // segs))))
    parts = segs * -(-quanta // per) * (Hq // Hkv)
    assert kve.decode_workspace_size(L, B, Hq, Hkv, N, d) == up(4 * parts * d) + up(8 * parts)
