"""How the batched launch hands out its claims (csrc/aes_batch_claims.hpp,
compiled here for the CPU): lists are played through the kernel's rules, a wave
busy for as many rows of 64 blocks as its item has, and must end about as early
as with every claim taken alone when a wave is free."""
import ctypes
import heapq
import os
import subprocess

import numpy as np
import pytest

from paper_1902_05234_amd import inputs

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_1902_05234_amd", "csrc")
WRAPPER = """
#include "aes_batch_claims.hpp"
extern "C" uint32_t dealt(uint32_t n, uint32_t waves, uint32_t worth)
{
    return aesgpu::claims_of(n, waves, worth).dealt;
}
extern "C" uint32_t claim_waves(uint32_t own, uint32_t all) { return aesgpu::claim_waves(own, all); }
extern "C" uint32_t claims_worth(uint64_t blocks, uint64_t n) { return aesgpu::claims_worth(blocks, n); }
extern "C" uint32_t at_once(uint32_t left, uint32_t waves, uint32_t taken, uint32_t longest, uint32_t worth)
{
    return aesgpu::claims_at_once(left, aesgpu::list_claims(0, waves, waves, 1).per_wave, taken, longest, worth);
}
extern "C" void short_list(uint64_t n_enc, uint64_t n_dec, uint32_t per_group, uint64_t max_grid, uint64_t resident,
                           uint32_t* out)
{
    const aesgpu::ShortList s = aesgpu::short_list(n_enc, n_dec, per_group, max_grid, resident);
    out[0] = s.parts_log2, out[1] = s.grid, out[2] = s.enc_groups;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("claims")
    (d / "w.cpp").write_text(WRAPPER)
    so = str(d / "w.so")
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC,
                        str(d / "w.cpp"), "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = ctypes.CDLL(so)
    lib.claims_worth.argtypes = [ctypes.c_uint64, ctypes.c_uint64]
    for f in (lib.dealt, lib.claim_waves, lib.claims_worth, lib.at_once):
        f.restype = ctypes.c_uint32
    return lib


def play(lists, groups, per_group, rules=None):
    """Time at which the last wave of `groups` = (on list 0, on list 1)
    workgroups is done with both lists; rules None: one claim at a time."""
    total = sum(groups) * per_group
    worth = rules.claims_worth(int(sum(map(np.sum, lists))), sum(map(len, lists))) if rules else 1
    dealt = [rules.dealt(len(x), g * per_group, worth) if rules else 0 for x, g in zip(lists, groups)]
    counter, times, done = [0, 0], [], [0, 0]
    heap = []  # (time, workgroup, wave) of waves that look for an item; state beside it
    state = {}
    finished = {}
    for wg in range(sum(groups)):
        own = 0 if wg < groups[0] else 1
        first = wg if own == 0 else wg - groups[0]
        for w in range(per_group):
            state[wg, w] = dict(list=own, at=first * per_group + w, run=0, taken=1, longest=0,
                                left=len(lists[own]) - dealt[own], next=0, second=False)
            heap.append((0.0, wg, w))
        finished[wg] = []
    heapq.heapify(heap)
    while heap:
        t, wg, w = heapq.heappop(heap)
        s = state[wg, w]
        k = s["list"]
        n = len(lists[k])
        if not s["second"] and s["at"] < dealt[k]:
            i = s["at"]
            s["at"] += groups[k] * per_group
        elif dealt[k] < n:
            if s["run"] == 0:
                r = 1
                if rules:
                    r = rules.at_once(s["left"], rules.claim_waves(groups[k] * per_group, total), s["taken"],
                                      s["longest"], worth)
                s["run"] = s["taken"] = r
                s["longest"] = 0
                s["next"] = dealt[k] + counter[k]
                counter[k] += r
                s["left"] = max(0, n - s["next"])
            i = s["next"]
            s["next"] += 1
            s["run"] -= 1
        else:
            i = n
        if i < n:
            done[k] += 1
            s["longest"] = max(s["longest"], int(lists[k][i]))
            heapq.heappush(heap, (t + -(-int(lists[k][i]) // 64), wg, w))
            continue
        finished[wg].append(t)
        if len(finished[wg]) == per_group:  # the workgroup meets, then helps or ends
            t = max(finished[wg])
            other = 1 - k
            left = len(lists[other]) - dealt[other] - counter[other]
            if s["second"] or left <= 0:
                times.append(t)
                continue
            finished[wg] = []
            for v in range(per_group):
                state[wg, v] = dict(list=other, at=0, run=0, taken=1, longest=0, left=left, next=0, second=True)
                heapq.heappush(heap, (t, wg, v))
    assert done == [len(x) for x in lists]
    return max(times)


def lists_of_very_unequal_size():
    g = inputs.rng(23)
    for few, many, length in ((1, 800, 256), (10, 5000, 256), (10, 5000, 64), (3, 20000, 16)):
        yield "%d and %d of %d" % (few, many, length), (np.full(few, length), np.full(many, length)), (1, 15)
        yield "%d long and %d of %d" % (few, many, length), (np.full(few, 2048), np.full(many, length)), (1, 15)
    yield "5 and 5000 of 1..256", (np.full(5, 8), g.integers(1, 257, 5000)), (1, 15)
    yield "3000 on one group, 40 on the others", (np.full(3000, 128), np.full(40, 128)), (1, 15)


def test_helpers_take_no_more_than_their_share(lib):
    for name, lists, groups in lists_of_very_unequal_size():
        alone = play(lists, groups, 16)
        longest = -(-max(int(x.max()) for x in lists) // 64)
        # a wave's last claims may hold a sixteenth of its share more than the others'
        assert play(lists, groups, 16, lib) <= 1.1 * alone + longest, name


def test_idle_waves_of_one_direction_find_claims_of_the_other(lib):
    """Workgroups split by item count, items of one direction long and of the
    other one block: with every wave's first claim dealt the long list still
    has claims for the waves that are through with the short one."""
    waves = 16 * 16
    for per_wave in (2, 3, 4, 5, 7, 10, 16, 40):
        n = per_wave * waves // 2
        lists = (np.full(n, 2048), np.ones(n, dtype=int))
        for pair in (lists, lists[::-1]):
            # as many rows more as the short list's items take
            assert play(pair, (8, 8), 16, lib) <= 1.1 * play(pair, (8, 8), 16) + per_wave, per_wave


@pytest.mark.parametrize("resident,per_group", [(256, 16), (512, 16), (4096, 1)])
def test_short_lists_take_no_more_workgroups_than_are_resident(lib, resident, per_group):
    """An explicit grid is a limit, not the device's size: parts of items are
    made for the waves that the device holds, one claim each."""
    out = (ctypes.c_uint32 * 3)()
    u64 = ctypes.c_uint64
    for n_enc, n_dec in ((1, 0), (0, 1), (7, 3), (500, 500), (0, 1000), (4000, 90), (4096, 0), (2048, 2049), (9000, 1)):
        for max_grid in (1, 2, 63, 256, 4096, 2**31 - 1):
            lib.short_list(u64(n_enc), u64(n_dec), per_group, u64(max_grid), u64(resident), out)
            lp, grid, enc_groups = out
            room = min(max_grid, resident)
            need = -(-n_enc // per_group) + -(-n_dec // per_group)
            assert (grid != 0) == (need <= room)
            if grid:
                assert grid <= room and lp <= 5
                assert (n_enc << lp) <= enc_groups * per_group and (n_dec << lp) <= (grid - enc_groups) * per_group
                more = -(-(n_enc << lp + 1) // per_group) + -(-(n_dec << lp + 1) // per_group)
                assert lp == 5 or more > room


def test_counter_does_not_wrap_where_single_claims_would_not(lib):
    """Every wave's last update may pass the end of the list, with what the wave
    thought was left at most the whole list."""
    for waves in (1, 16, 4096, 16 * 1024):
        for n in (1000, 2**20, 2**30, 2**31 - 1, 2**31, 3 * 2**30, 2**32 - 2**20, 2**32 - 1):
            for blocks in (0, n, 100 * n):
                worth = lib.claims_worth(blocks, n)
                most = max(lib.at_once(n, waves, taken, longest, worth) for taken in (1, 2**20) for longest in (1, 10**6))
                assert most <= worth
                assert worth == 1 or n + waves * most < 2**32, (waves, n, blocks)
