"""Host-side replay of the fused batched forward's index arithmetic (CPU only).

The library's host half is built with its kernel launchers replaced by one that
prints the plan a launch receives (tests/hostcheck/plan_driver.cpp), and the
kernels' index arithmetic is replayed on it over sampling intervals, orders,
generations, groups, tiles and segments:

* filters and polynomials (batch_kernels.hpp): a run of the projection leaves the
  workgroup's lanes room for the spread of the nine positions; every tap of the
  filters lies in a row its tile has written, and every interpolation the taps
  stand for lies within them; the 16 lanes of a row of output pairs read one
  table; the carried halo is what the next tile expects;
* delay by delay (batch_stream_kernels.hpp): the same for the stencils of single
  delays, and the window of h+ and hx fits the rows it borrows;
* which of the two runs, on both sides of the measured line.
"""
import json
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2204_06633_amd.csrc import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HC = os.path.join(ROOT, "tests", "hostcheck")


def _hipcc():
    for c in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if c and os.path.exists(c):
            return c
    return None


pytestmark = pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
ARM = 8.4
SIZES = [3000, 1, 33, 481, 0, 2999, 1400]


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("plan")
    csrc = os.path.join(ROOT, "paper_2204_06633_amd", "csrc")
    cc = [_hipcc(), "-O1", "-std=c++17", "--offload-arch=gfx950",
          "-I" + os.path.join(ROOT, "include")]
    objs = []
    for src, extra in ((os.path.join(HC, "plan_driver.cpp"), []),
                       (os.path.join(HC, "launch_stubs.cpp"),
                        ["-D%s=unused_%s" % (f, f)
                         for f in ("run_fused_forward", "run_tdi", "run_tdi_adjoint")]),
                       (os.path.join(csrc, "api.cpp"), []), (os.path.join(csrc, "api_batch.cpp"), [])):
        objs.append(str(tmp / (os.path.basename(src) + ".o")))
        subprocess.check_call(cc + extra + ["-c", src, "-o", objs[-1]], stderr=subprocess.DEVNULL)
    exe = str(tmp / "plan")
    subprocess.check_call(cc + objs + ["-o", exe] + build.link_flags(), stderr=subprocess.DEVNULL)

    def run(cases):
        """cases: (order, gen, dt, projection arm, TDI arm, group, tile, segment, sizes)
        of a batch, or (order, gen, dt, arm, outputs) of a TDI call."""
        text = "".join("tdi %d %d %r %r %d\n" % c if len(c) == 5 else
                       "batch %d %d %r %r %r %d %d %d %d %s\n"
                       % (*c[:8], len(c[8]), " ".join(map(str, c[8]))) for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=300)
        assert out.returncode == 0, out.stderr
        return [json.loads(line) for line in out.stdout.splitlines()]
    return run


def _halo_cap(group, lanes):
    c = (2 * lanes // (6 * group)) & ~1
    return 0 if c < 32 else min(c, 64)


def _replay(case, p):
    order, gen, dt, arm_p, arm_t, group, tile, segment, sizes = case
    N, H, lanes, chain = order + 1, (order + 1) // 2, tile // 2, 3 if gen == 1 else 7
    hp, K, lo, F = p["HP"], p["fir_k"], p["fir_lo"], p["F"]
    row_len = tile + _halo_cap(group, lanes)
    assert hp in (0, p["halo"]) and hp <= _halo_cap(group, lanes)
    assert p["T_out"] >= 2 and p["T_out"] + p["halo"] <= p["samples"] <= tile
    spread = int(np.ceil(2.01 * max(arm_p, arm_t) / dt)) + 2
    shifts = np.floor(-np.linspace(0.98 * arm_t, chain * arm_t, 1001) / dt).astype(int)
    if K:
        assert p["rows"] + spread <= lanes, "a run's positions outgrow the workgroup's bases"
        assert shifts.min() - (H - 1) >= lo and shifts.max() + H <= lo + K - 1
        assert lo <= 0 <= lo + K - 1                       # the undelayed terms
        assert p["n_fir"] * 512 >= max(sizes)
    else:
        assert p["samples"] == tile == p["T_out"] + p["halo"]
        if max(arm_p, arm_t) <= 1.25 * arm_t:
            assert tile + spread + N + 1 <= 3 * row_len, "the window outgrows its rows"
    groups = -(-len(sizes) // group)
    longest = [sorted(sizes, reverse=True)[g * group] for g in range(groups)]
    seen = [np.zeros(n, int) for n in longest]
    seg_out = p["T_out"] + (p["tiles"] - 1) * p["samples"]
    for g, seg in p["items"]:
        assert seg * seg_out < longest[g]
        link = None                                        # link sample of each row
        for t in range(p["tiles"]):
            o0 = seg * seg_out + (0 if t == 0 else p["T_out"] + (t - 1) * p["samples"])
            if o0 >= longest[g]:
                break
            cnt, ro = (p["T_out"], hp) if t == 0 else (p["samples"], 0)
            rows = np.full(row_len + 1, -10 ** 9)
            if t > 0:                                      # the carried halo
                at = hp + p["T_out"] if t == 1 else p["samples"]
                rows[:hp] = link[at:at + hp]
            rows[hp:hp + p["samples"]] = o0 - F + (0 if t == 0 else hp) + np.arange(p["samples"])
            oa = 2 * np.arange(lanes) - (o0 % 32 if K else 0)
            ob = np.clip(oa, 0, cnt - 2)
            done = oa[(oa >= 0) & (oa < cnt)]
            assert np.array_equal(np.sort(np.r_[done, done + 1]), np.arange(cnt))
            if K:
                # row of tap k of output o0 + ob: link sample o0 + ob + lo + k, and
                # one more for the pair's second output
                for k in (0, K - 1, K):
                    assert np.array_equal(rows[F + lo + ro + ob + k], o0 + ob + lo + k)
                q = (o0 + ob) // 512
                assert (q.reshape(-1, 16) == q.reshape(-1, 16)[:, :1]).all()
            else:
                for s in (shifts.min() - (H - 1), shifts.max() + H + 1, 0, 1):
                    assert np.array_equal(rows[F + ro + ob + s], o0 + ob + s)
                assert F + ro + ob.max() + shifts.max() - (H - 1) <= row_len - 1 - N
            n = min(cnt, longest[g] - o0)
            seen[g][o0:o0 + n] += 1
            link = rows
    assert all((s == 1).all() for s in seen)


@pytest.mark.parametrize("gen", [1, 2])
@pytest.mark.parametrize("order", [1, 7, 13, 25, 31])
def test_work_items_replayed(plans, order, gen):
    todo = [(order, gen, dt, arm, ARM, group, tile, segment, SIZES)
            for dt in (0.4, 0.7, 1.0, 1.3, 1.7, 2.5, 5.0, 10.0, 15.0, 60.0)
            for group in (1, 2, 4) for tile in (256, 512, 1024) if (group, tile) != (4, 1024)
            for segment in (0, 3) for arm in (ARM, 1.2 * ARM, 40.0)]
    done = 0
    for case, p in zip(todo, plans(todo)):
        if p["workspace"] == 0:                            # the TDI halo does not fit the tile
            continue
        # the workspace, sized without the projection's orbits, suffices for any
        assert p["status"] == 0, case
        _replay(case, p)
        done += 1
    assert done > 250


# (order, generation, dt, filters), 32 templates of 60,000 outputs in groups of two, us
# delay by delay and with filters: beside each line
ROUTES = [(1, 1, 10.0, False),      # 111, 130
          (3, 1, 10.0, False),      # 131, 132; synthesised 131, 144
          (7, 1, 10.0, True),       # 158, 155
          (7, 1, 5.0, False),       # 156, 178
          (13, 1, 5.0, True),       # 209, 204
          (25, 1, 5.0, True),       # 299, 259
          (25, 1, 1.0, False),      # 336, 346
          (1, 2, 10.0, True),       # 140, 132
          (1, 2, 5.0, False),       # 142, 150
          (3, 2, 5.0, True),        # 225, 165
          (25, 2, 10.0, True),      # 416, 255
          (25, 2, 2.5, True),       # 484, 363
          (7, 2, 1.5, False),       # 253, 269 (synthesised)
          (25, 2, 1.0, False),      # 554, 669 (groups of one)
          (25, 2, 0.7, False)]      # 566, 611


@pytest.mark.parametrize("order,gen,dt,filters", ROUTES)
def test_filters_only_where_they_are_faster(plans, order, gen, dt, filters):
    case = (order, gen, dt, ARM, ARM, 2, 512, 0, [200000])
    bare = (order, gen, dt, ARM, ARM, 2, 512, 0, [1])
    p, q = plans([case, bare])
    assert (p["fir_k"] > 0) == filters
    # 48 B of link gradients and some of work lists per output; tables of up to 60 B
    assert p["workspace"] - q["workspace"] < (52 + (60 if filters else 1)) * 200000


def test_longer_projection_arms_leave_the_filters(plans):
    """Runs are sized by the TDI's light times: projection orbits that spread the
    positions further take the kernel whose window holds them."""
    for arm, filters in ((ARM, True), (1.2 * ARM, True), (1.7 * ARM, False), (40.0, False)):
        p, = plans([(25, 2, 2.0, arm, ARM, 2, 512, 0, SIZES)])
        assert (p["fir_k"] > 0) == filters, arm


# (order, generation, dt, outputs, filters forward, transpose): us one by one and with
# filters beside each line
TDI_ROUTES = [(1, 2, 2.5, 200000, False, True),        # 21.1, 23.8; 36.7, 27.3
              (3, 1, 5.0, 1600000, False, True),       # 56.8, 60.8; 126, 74
              (7, 1, 1.0, 200000, False, False),       # 18.7, -; 30.8, 34.0
              (7, 1, 10.0, 1600000, True, True),       # 72.7, 62.1; 125.6, 74.1
              (7, 1, 1.0, 1600000, False, False),      # 72.9, -; 128, 127 (filters by count 149)
              (25, 1, 1.0, 1600000, False, True),      # 136, -; 264, 205
              (1, 2, 5.0, 1600000, True, True),        # 72.3, 66.6; 136, 76.7
              (7, 2, 2.5, 1600000, True, True),        # 124.8, 124.3; 185.7, 130.6
              (25, 2, 1.55, 1600000, True, True),      # 302, 244; 480, 262
              (25, 2, 10.0, 8640, True, True),         # 25, 17; 76, 24
              (1, 1, 10.0, 8640, True, True),          # 12, 10; 27, 15
              (25, 2, 1.0, 1600000, False, False)]     # too many taps for LDS


@pytest.mark.parametrize("order,gen,dt,n,forward,transpose", TDI_ROUTES)
def test_tdi_filters_only_where_they_are_faster(plans, order, gen, dt, n, forward, transpose):
    p, = plans([(order, gen, dt, ARM, n)])
    assert (p["forward"] > 0, p["transpose"] > 0) == (forward, transpose)
