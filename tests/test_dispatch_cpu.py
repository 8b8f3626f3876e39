"""Which kernels the calls launch, without a GPU: the library runs on a stand-in for the HIP runtime that writes the
launches down (hip_recorder.cpp), in a process of its own."""
import json
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, json, sys
sys.path.insert(0, {root!r})
rec = ctypes.CDLL({recorder!r}, mode=ctypes.RTLD_GLOBAL)        # found before the real runtime
rec.recorder_name.restype = ctypes.c_char_p
rec.recorder_grid.restype = ctypes.c_uint
from paper_1904_04956_amd import binding as bl
P = 1 << 20                                                      # any aligned address: nothing is read or written


class Model:
    def __init__(self, mode=1, **dims):
        self.ctx = bl.blstm_create(mode=mode, **dims)
        bl.blstm_bind(self.ctx, P, bl.blstm_workspace_bytes(self.ctx))
    def option(self, which, value): bl.blstm_set_option(self.ctx, which, value)
    def forward(self, stream=0): bl.blstm_forward(self.ctx, P, P, P, stream)
    def xent(self, stream=0): bl.softmax_xent_fwd_bwd(self.ctx, P, P, P, P, P, P, stream)
    def noalloc(self, stream=0): bl.softmax_xent_fwd_bwd_noalloc(self.ctx, P, P, P, P, P, P, stream)
    def backward(self, stream=0): bl.blstm_backward(self.ctx, P, P, P, P, stream)


def launches(call):
    rec.recorder_clear()
    call()
    return [rec.recorder_name(i).decode() for i in range(rec.recorder_count())]


def count(names, part): return sum(part in n for n in names)
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    out = str(tmp_path_factory.mktemp("recorder") / "librecorder.so")
    subprocess.run([gxx, "-O1", "-shared", "-fPIC", "-std=c++17", "-o", out, os.path.join(HERE, "hip_recorder.cpp")], check=True)

    def run(code):
        text = PRELUDE.format(root=ROOT, recorder=out) + textwrap.dedent(code) + "\nprint(json.dumps(out))\n"
        r = subprocess.run([sys.executable, "-c", text], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout.splitlines()[-1])
    return run


DIMS = "T=4, B=16, D=8, H=640, L=2, P=0, V=20"             # 80 workgroups of the small kernels, wider than the ones that fill


def test_exchange_copies_count_as_marked_only_if_the_launched_kernels_marked_them(recorder):
    # where the kernels for few sequences do not fit, those of recurrent.hip run: at this width they mark nothing
    small, large = recorder(f"""
        out = []
        for device, small_fits in ((0, 1), (1, 0)):
            rec.recorder_device(device)
            rec.recorder_occupancy(b"rec_small", small_fits)
            m = Model({DIMS})
            f, b = launches(m.forward), launches(m.backward)
            out.append([count(f, "rec_small_fwd"), count(f, "14rec_fwd_kernel"), count(b, "rec_small_bwd"), count(b, "14rec_bwd_kernel"), count(b, "fill_u128")])
    """)
    assert small == [2, 0, 2, 0, 0]
    assert large == [0, 2, 0, 2, 1]


@pytest.mark.parametrize("dims,fwd,bwd,other", [             # (mangled names: tile_rec_fwd_kernel contains rec_fwd_kernel)
    (DIMS, "rec_small_fwd", "rec_small_bwd", "14rec_fwd_kernel"),
    ("T=4, B=600, D=8, H=512, L=1, P=0, V=20", "tile_rec_fwd", "tile_rec_bwd", "cell_fwd"),
    ("T=4, B=40, D=8, H=1024, L=1, P=0, V=20", "tile_rec_fwd", "tile_rec_bwd", "14rec_fwd_kernel"),
    ("T=4, B=2100, D=8, H=96, L=1, P=0, V=20", "14rec_fwd_kernel", "14rec_bwd_kernel", "cell_fwd"),
])
def test_a_forward_kernel_runs_only_if_its_backward_twin_fits_too(recorder, dims, fwd, bwd, other):
    f_twin, f_other, b_twin = recorder(f"""
        rec.recorder_occupancy(b"rec_", 2)
        rec.recorder_occupancy(b"{bwd}", 0)
        m = Model({dims})
        f = launches(m.forward)
        b = launches(m.backward)
        out = [count(f, "{fwd}"), count(f, "{other}"), count(b, "{bwd}")]
    """)
    assert f_twin == 0 and f_other > 0 and b_twin == 0


@pytest.mark.parametrize("mode,dims", [(1, "T=4, B=16, D=8, H=512, L=1, P=0, V=20"), (1, "T=4, B=256, D=8, H=512, L=1, P=0, V=20"),
                                       (0, "T=4, B=64, D=8, H=512, L=1, P=0, V=20")])
def test_whether_a_grid_fits_is_asked_for_every_device(recorder, mode, dims):
    big, little, big_again = recorder(f"""
        rec.recorder_cus(1, 16)
        out = []
        for device in (0, 1, 0):
            rec.recorder_device(device)
            m = Model(mode={mode}, {dims})
            f = launches(m.forward)
            out.append([count(f, "rec_small_fwd") + count(f, "tile_rec_fwd") + count(f, "rec32_fwd"), count(f, "cell_fwd")])
    """)
    assert big == big_again == [1, 0]
    assert little == [0, 4]


def test_learners_of_several_batches_do_not_ask_again_what_fits(recorder):
    # the LDS of their kernels differs, by the tiles a workgroup keeps the state of; two devices
    first, again = recorder("""
        rec.recorder_occupancy(b"rec_", 2)
        made = [[Model(T=2, B=B, D=8, H=512, L=1, P=0, V=20) for B in (600, 1200)] for device in (0, 1)]
        out, last = [], 0
        for k in range(4):
            for device in (0, 1):
                rec.recorder_device(device)
                for m in made[device]: m.forward(); m.backward()
            out.append(rec.recorder_occupancy_asked() - last)
            last += out[-1]
        out = [out[0], sum(out[1:])]
    """)
    assert first > 0 and again == 0


@pytest.mark.parametrize("dims", [DIMS, "T=4, B=256, D=8, H=1024, L=1, P=0, V=20", "T=4, B=600, D=8, H=512, L=2, P=0, V=20", "T=4, B=70, D=30, H=101, L=1, P=0, V=20",
                                  "mode=0, T=4, B=64, D=8, H=512, L=2, P=0, V=20", "mode=0, T=4, B=64, D=8, H=101, L=2, P=301, V=9001"])
def test_a_captured_backward_pass_marks_what_its_replays_exchange(recorder, dims):
    # marked by the forward pass only where both are launched, or both are in one graph
    fills = recorder(f"""
        rec.recorder_occupancy(b"rec_", 4)
        m = Model({dims})
        fills = lambda s: count(launches(lambda: m.backward(s)), "fill_u128")
        graph, other = 1 << 16, 1 << 17
        out = []
        m.forward(); out.append(fills(0))
        m.forward()
        rec.recorder_capturing(ctypes.c_void_p(graph)); out.append(fills(graph))      # behind a launched one
        rec.recorder_capturing(ctypes.c_void_p(graph)); m.forward(graph); out.append(fills(graph)); out.append(fills(graph))
        m.forward(graph); rec.recorder_capturing(ctypes.c_void_p(graph)); out.append(fills(graph))   # in a graph of its own
        m.forward(graph); rec.recorder_capturing(None); out.append(fills(0))
    """)
    assert fills == [0, 1, 0, 1, 1, 1]


@pytest.mark.parametrize("mode,dims", [(1, DIMS), (1, "T=4, B=600, D=8, H=512, L=2, P=0, V=20"), (1, "T=4, B=70, D=30, H=101, L=1, P=0, V=20"),
                                       (0, "T=4, B=64, D=8, H=512, L=2, P=0, V=20"), (0, "T=4, B=64, D=8, H=101, L=2, P=301, V=9001")])
@pytest.mark.parametrize("with_forward", [False, True])
def test_a_backward_pass_marks_its_copies_where_a_replay_may_have_written_them(recorder, mode, dims, with_forward):
    # a graph with a backward pass is there; then forward, (its replay, which no call shows,) backward: what the forward pass marked may be the replay's
    # dE/da by now, which would be taken for this pass's
    before, captured, after = recorder(f"""
        rec.recorder_occupancy(b"rec", 4)
        m = Model({mode}, {dims})
        fills = lambda s: count(launches(lambda: m.backward(s)), "fill_u128")
        graph = 1 << 16
        m.forward(); out = [fills(0)]
        m.forward()
        rec.recorder_capturing(ctypes.c_void_p(graph))
        if {with_forward}: m.forward(graph)
        out.append(fills(graph))
        rec.recorder_capturing(None)
        m.forward(); out.append(fills(0))
    """)
    assert [before, captured, after] == [0, 0 if with_forward else 1, 1]


@pytest.mark.parametrize("B,H,one", [(64, 512, True), (8, 768, True), (150, 512, False), (512, 512, False), (30, 772, False), (30, 1024, False)])
def test_float_exchange_copies_are_per_layer_only_where_the_forward_kernel_marks_them(recorder, B, H, one):
    # fills of a forward and of a backward pass, the same behind another backward pass, and what a layer more adds to the workspace
    fills, grown = recorder(f"""
        out, bytes = [], []
        for L in (2, 3):
            m = Model(mode=0, T=4, B={B}, D=8, H={H}, L=L, P=0, V=20)
            bytes.append(bl.blstm_workspace_bytes(m.ctx))
            out += [count(launches(call), "fill_u128") for call in (m.forward, m.backward, m.backward)]
        out = [out, bytes[1] - bytes[0]]
    """)
    up, T = lambda n, m: (n + m - 1) // m * m, 4               # noqa: E731
    rows, kept = T * up(B, 32), 4 * up(H, 32)
    layer = up(T * B * 2 * H * 4, 256) + up(rows * 8 * kept, 256) + up(rows * 2 * kept, 256) + up(T * B * 8 * H * 4, 256)   # y, gates, c, dE/da
    copies = T * 2 * up(B, 32) // 32 * up(H, 8) // 8 * 1024 + T * 2 * up(B, 16) // 16 * up(H, 16) // 16 * 4096
    assert fills == ([1, 0, 1] * 2 if one else [2, 2, 2, 3, 3, 3])
    assert grown == layer + (copies if one else 0)


@pytest.mark.parametrize("dims,copy,axis", [("T=4, B=16, D=8, H=101, L=2, P=0, V=20", "pad_blocks", 0),      # a twin's weights
                                            ("T=4, B=16, D=30, H=104, L=2, P=0, V=20", "pad_cols", 1)])        # W_x of the first layer
def test_a_weight_copy_that_failed_is_made_again(recorder, dims, copy, axis):
    # with copies kept from call to call: a failed launch leaves none behind
    failed, again, kept = recorder(f"""
        m = Model({dims})
        m.option(bl.BLSTM_OPT_KEEP_WEIGHT_COPIES, 1)
        rec.recorder_fail(b"{copy}")
        out = []
        try:
            m.forward()
        except bl.BlstmError as e:
            out.append(e.code)
        rec.recorder_fail(b"")
        for _ in range(2):
            n = launches(m.forward)
            out.append([rec.recorder_grid(i, 1) if {axis} else 1 for i in range(len(n)) if "{copy}" in n[i]])   # (x and the two directions' weights, or x alone)
    """)
    assert failed == -5
    assert again == [3] if axis else again == [1]
    assert kept == [1] if axis else kept == []


@pytest.mark.parametrize("mode,dims", [(1, "T=4, B=16, D=8, H=104, L=2, P=0, V=20"), (1, "T=4, B=16, D=30, H=101, L=2, P=37, V=20"),
                                       (0, "T=21, B=16, D=33, H=66, L=2, P=301, V=9001")])
def test_profiling_times_every_launch(recorder, mode, dims):
    n_launches, untimed, calls, n_timed = recorder(f"""
        m = Model(mode={mode}, {dims})
        out = [0, [], 0, 0]
        bl.lib().blstm_profile_enable(m.ctx, 1)
        for call in (m.forward, m.xent, m.noalloc, m.backward):
            n = launches(call)
            out[0] += len(n)
            out[1] += [n[i] for i in range(len(n)) if not rec.recorder_timed(i)]
            out[2] += 1
        k = bl.lib().blstm_profile_classes()
        ms, count = (ctypes.c_double * k)(), (ctypes.c_int64 * k)()
        bl.lib().blstm_profile_read(m.ctx, ms, count, k)
        out[3] = sum(count)
    """)
    assert calls == 4 and untimed == []
    assert 0 < n_timed <= n_launches                       # (one pair of events may hold several launches)


@pytest.mark.parametrize("models,streams,together", [
    ([(1, 256, 512)], [256, 512], 256),                    # (mode, sequences, cells); each launch fills the device
    ([(0, 64, 512)], [256, 512], 256),
    ([(1, 16, 512), (0, 16, 64), (1, 40, 101)], [256, 512, 768], None),
    ([(1, 16, 512)], [256, 512, 768, 1024, 0], 256),        # 64 workgroups a launch: four fit, the fifth waits
    ([(1, 8, 128)], [256 * k for k in range(1, 13)], 128),  # more streams than lanes: eight of 16 workgroups
    ([(1, 256, 512), (1, 16, 512), (1, 2000, 256), (1, 8, 128)], [256, 512, 768], None),   # every stream goes from large launches to small ones and back
])
def test_persistent_launches_that_may_run_at_once_fit_the_device(recorder, models, streams, together):
    # their workgroups wait on each other: grids that are not ordered never have more than the device's 256 CUs together
    grids, behind, captured = recorder(f"""
        made = [[Model(mode=m, T=4, B=B, D=8, H=H, L=2, P=0, V=20) for m, B, H in {models}] for s in {streams}]
        for k in range({len(models)} + 1):
            for i, s in enumerate({streams}):
                m = made[i][(i + k) % {len(models)}]
                m.forward(s); m.xent(s); m.backward(s)
        n = rec.recorder_persistent()
        out = [[rec.recorder_workgroups(i) for i in range(n)], [[rec.recorder_behind(i, j) for j in range(i)] for i in range(n)]]
        rec.recorder_capturing(ctypes.c_void_p(1 << 16))   # (launched without events: nothing a capture refuses)
        out.append(count(launches(lambda: made[0][0].forward(1 << 16)), "rec"))
    """)
    assert captured == 2 and all(g % 8 == 0 for g in grids)
    small = [i for i in range(len(grids)) if grids[i] <= 256]
    worst = _most_at_once([grids[i] for i in small], [[behind[i][j] for j in small if j < i] for i in small])
    assert worst <= 256 and (together is None or worst == together)
    assert _most_at_once(grids, behind) <= max(256, max(grids))   # (a larger one runs alone)


def test_idle_streams_keep_nobody_waiting(recorder):
    # five streams ran something earlier; three that fit the device together still run side by side
    last, ordered = recorder("""
        made = [Model(T=4, B=16, D=8, H=512, L=1, P=0, V=20) for s in range(8)]
        for m, s in zip(made, range(1, 9)): m.forward(256 * s)
        for k in range(3):
            for s in (6, 7, 8): made[s - 1].forward(256 * s)
        n = rec.recorder_persistent()
        out = [[rec.recorder_workgroups(i) for i in range(n - 3, n)], [rec.recorder_behind(i, j) for i in range(n - 3, n) for j in range(n - 3, i)]]
    """)
    assert last == [64, 64, 64] and ordered == [0, 0, 0]


def _most_at_once(weight, behind):
    # the heaviest set of launches none of which is behind another: the least flow through the order that gives every launch its weight
    from scipy.optimize import linprog
    from scipy.sparse import lil_matrix
    n = len(weight)
    edges = [(j, i) for i in range(n) for j in range(i) if behind[i][j]]
    into, outof = lil_matrix((n, 2 * n + len(edges))), lil_matrix((n, 2 * n + len(edges)))
    for i in range(n):
        into[i, i] = outof[i, n + i] = 1.0
    for k, (j, i) in enumerate(edges):
        outof[j, 2 * n + k] = into[i, 2 * n + k] = 1.0
    cost = [1.0] * n + [0.0] * (n + len(edges))
    r = linprog(cost, A_ub=-into.tocsr(), b_ub=[-w for w in weight], A_eq=(into - outof).tocsr(), b_eq=[0.0] * n, method="highs")
    assert r.status == 0
    return round(r.fun)


@pytest.mark.parametrize("B,H,fwd,bwd", [
    (64, 512, True, True), (256, 256, True, True), (4096, 64, True, True), (15, 1024, True, True),
    (1408, 576, False, False), (1280, 704, False, False), (1024, 768, False, False), (4096, 384, False, False),   # were persistent, and slower for it
    (384, 704, True, False), (8192, 128, True, False), (4096, 200, True, False),
    (768, 1024, True, False), (2048, 512, True, False),
])
def test_float_recurrences_take_the_faster_path(recorder, B, H, fwd, bwd):
    f, b = recorder(f"""
        m = Model(mode=0, T=2, B={B}, D=8, H={H}, L=1, P=0, V=20)
        f, b = launches(m.forward), launches(m.backward)
        out = [[count(f, "rec32_fwd"), count(f, "cell_fwd")], [count(b, "rec32_bwd"), count(b, "cell_bwd")]]
    """)
    assert f == ([1, 0] if fwd else [0, 2]) and b == ([1, 0] if bwd else [0, 2])


@pytest.mark.parametrize("B,H,persistent", [(3072, 576, True), (3073, 576, False), (4096, 768, False), (16384, 504, True), (4096, 1024, True)])
def test_padded_widths_of_many_sequences_take_the_faster_path(recorder, B, H, persistent):
    f, b = recorder(f"""
        m = Model(T=2, B={B}, D=8, H={H}, L=1, P=0, V=20)
        out = [[count(n, "rec_fwd") + count(n, "rec_bwd"), count(n, "cell_")] for n in (launches(m.forward), launches(m.backward))]
    """)
    assert f == b == ([1, 0] if persistent else [0, 2])


@pytest.mark.parametrize("mode,H,T,persistent", [(1, 320, 1, False), (1, 320, 2, True), (1, 512, 1, True), (0, 32, 1, False), (0, 32, 2, True)])
def test_a_single_frame_needs_no_recurrence(recorder, mode, H, T, persistent):
    # (of bf16 widths with kernels of their own the one launch is as short as the cell's)
    f, b = recorder(f"""
        m = Model(mode={mode}, T={T}, B=16, D=8, H={H}, L=1, P=0, V=20)
        out = [[count(n, "rec"), count(n, "cell_")] for n in (launches(m.forward), launches(m.backward))]
    """)
    assert f == b == ([1, 0] if persistent else [0, 1])


@pytest.mark.parametrize("mode,dims,parts", [
    (1, "T=20, B=23, D=40, H=128, L=1, P=461, V=2000", 8),     # z's rows are unaligned, and the model too small for a twin
    (1, "T=20, B=23, D=40, H=128, L=1, P=66, V=1500", 6),
    (1, "T=20, B=23, D=40, H=101, L=1, P=0, V=2000", 8),       # the workspace form runs on the twin's aligned operands
    (1, "T=20, B=16, D=40, H=512, L=3, P=461, V=4000", 13),
    (0, "T=20, B=23, D=40, H=128, L=1, P=461, V=2000", None),
    (0, "T=20, B=28, D=40, H=256, L=3, P=250, V=2000", None),
])
def test_guarded_products_keep_their_parts(recorder, mode, dims, parts):
    # dz and dW_s of a model whose rows of z are unaligned, by either entry point: parts for 128x128 tiles, the only guarded ones
    forms = recorder(f"""
        out = []
        m = Model(mode={mode}, {dims})
        for call in (m.xent, m.noalloc):
            names = launches(call)
            out.append([rec.recorder_grid(i, 1) for i in range(len(names)) if "gemm_kernel" in names[i]])
    """)
    assert forms[0] == forms[1] and len(forms[0]) == 3
    assert forms[0][1] > 1 if parts is None else forms[0][1] == parts


@pytest.mark.parametrize("B,H,units,fwd,bwd", [
    (2048, 24, 2, 256, 256), (2049, 24, 2, 264, 264), (4097, 32, 2, 520, 520), (8193, 8, 2, 344, 344),   # up to four a CU, beyond that two with several tiles
    (2048, 64, 4, 256, 256), (2049, 64, 4, 264, 264), (4097, 64, 4, 176, 176),
    (1025, 128, 4, 272, 272), (513, 256, 4, 288, 160),       # the backward kernel fits a CU once
    (640, 136, 4, 240, 240), (641, 136, 2, 440, 440), (769, 136, 4, 312, 168),
])
def test_workgroups_on_sixteen_row_tiles(recorder, B, H, units, fwd, bwd):
    got = recorder(f"""
        rec.recorder_occupancy(b"tile_rec", 4)
        m = Model(T=2, B={B}, D=8, H={H}, L=1, P=0, V=20)
        out = []
        for call in (m.forward, m.backward):
            names = launches(call)
            out += [[names[i].split("kernelILi")[1][0], rec.recorder_grid(i, 0)] for i in range(len(names)) if "tile_rec" in names[i]]
    """)
    assert got == [[str(units), fwd], [str(units), bwd]]


@pytest.mark.parametrize("B,H,fwd,bwd", [
    (500, 256, True, True), (300, 256, True, True), (640, 136, True, True),     # <4, 8>
    (256, 512, False, False), (128, 512, False, False), (250, 256, True, False),
    (700, 136, True, True), (400, 264, True, True), (1500, 128, True, True),    # more than one workgroup a CU
    (190, 320, False, False), (1000, 128, False, True),
])
def test_sixteen_row_tiles_that_exchange_through_the_l2(recorder, B, H, fwd, bwd):
    got = recorder(f"""
        rec.recorder_occupancy(b"tile_rec", 4)
        m = Model(T=2, B={B}, D=8, H={H}, L=1, P=0, V=20)
        out = [[n.split("EEEv")[0][-1] for n in launches(call) if "tile_rec" in n] for call in (m.forward, m.backward)]
    """)
    assert got == [[str(int(fwd))], [str(int(bwd))]]


@pytest.mark.parametrize("B,H,asks", [(64, 512, True), (49, 392, True), (48, 512, False), (8, 512, False), (64, 384, False), (15, 1024, False), (30, 1024, False), (40, 640, False)])
def test_few_sequences_ask_for_their_xcd_only_where_groups_are_whole(recorder, B, H, asks):
    # (kernels that ask are those with NEAR set; contiguous eighths of the grid are whole groups where there are eight of them)
    (name,) = recorder(f"""
        m = Model(T=2, B={B}, D=8, H={H}, L=1, P=0, V=20)
        launches(m.forward)
        out = [n for n in launches(m.backward) if "rec_small_bwd" in n]
    """)
    assert name.split("EEEv")[0].endswith("ELb1" if asks else "ELb0")


@pytest.mark.parametrize("B,H,narrow", [(2048, 96, False), (2049, 96, True), (4096, 104, False), (4096, 64, False), (1280, 136, False), (1281, 160, True),
                                        (1025, 200, True), (1152, 288, False), (1153, 264, True), (4096, 328, False)])
def test_widths_with_an_empty_half_of_their_last_slice(recorder, B, H, narrow):
    # the forward kernel of recurrent.hip that marks dE/da's exchange copies on the side runs these
    f, b = recorder(f"""
        rec.recorder_occupancy(b"rec_", 4)
        m = Model(T=2, B={B}, D=8, H={H}, L=1, P=0, V=20)
        out = [[count(n, "14rec_fwd") + count(n, "14rec_bwd"), count(n, "tile_rec_"), count(n, "fill_u128")] for n in (launches(m.forward), launches(m.backward))]
    """)
    assert f == ([1, 0, 1] if narrow else [0, 1, 1]) and b == ([1, 0, 0] if narrow else [0, 1, 0])


GEMM = """
        def products(call):
            names = launches(call)
            return [[names[i].split("kernelI")[1].split("EEE")[0], rec.recorder_grid(i, 0), rec.recorder_grid(i, 1)] for i in range(len(names)) if "gemm_kernel" in names[i]]
"""


def test_tiles_of_the_products_that_are_checked_band_by_band(recorder):
    # the tile heights and rows that test_gpu_bands.py names
    from test_gpu_bands import BANDS
    got = recorder(GEMM + f"""
        out = []
        for M, D, H, *_ in {BANDS}:
            m = Model(T=1, B=M, D=D, H=H, L=1 if D > 24 else 2, P=0, V=20)
            out.append([p for p in products(m.forward) if p[0].startswith("tfLb0ELb0")][0])
    """)
    for (M, D, H, height, rows, band), (name, grid, parts) in zip(BANDS, got):
        tm, tn, wn = (int(c) for c in name.split("ELi")[1:4])   # (two wavefronts down, wn across, of tm x tn tiles of 32 x 32)
        assert (64 * tm, (M + 64 * tm - 1) // (64 * tm), parts) == (height, rows, 1)
        assert grid == rows * ((4 * H + 32 * tn * wn - 1) // (32 * tn * wn))
        assert band == (8 if M > 16384 and D * 4 * H * 2 <= 12 << 20 else 4)


@pytest.mark.parametrize("B,H,tiles", [(32, 1024, 96), (79, 1024, 208), (100, 512, 136)])
def test_input_gradients_with_a_long_contraction_are_split(recorder, B, H, tiles):
    # 128x128 tiles in two or more parts: unsplit on smaller tiles these took 1.2 to 1.6 times as long
    (dx,) = recorder(GEMM + f"""
        m = Model(T=21, B={B}, D=8, H={H}, L=2, P=0, V=20)
        launches(m.forward)
        out = products(m.backward)
    """)
    assert dx[0].startswith("tfLb0ELb1ELi2ELi2ELi2E") and dx[1] == tiles and dx[2] >= 2


@pytest.mark.parametrize("M,tile,grid,parts", [
    (16384, "tfLb0ELb1ELi4ELi2ELi4E", 64, 4),                 # 256x256, up to one workgroup per CU
    (16385, "tfLb0ELb1ELi2ELi2ELi2E", 258, 4),                # 65 of them fill no whole rounds
    (21021, "tfLb0ELb1ELi4ELi2ELi4E", 83, 3), (61184, "tfLb0ELb1ELi4ELi2ELi4E", 239, 2),   # whole rounds of them
    (61185, "ttLb0ELb1ELi4ELi2ELi2E", 480, 1),                # 256x128, unsplit
])
def test_tiles_and_parts_of_dz(recorder, M, tile, grid, parts):
    dz = recorder(GEMM + f"""
        out = [p for p in products(Model(T=1, B={M}, D=8, H=8, L=1, P=256, V=13001).xent) if "Lb0ELb1" in p[0]][0]   # (the dA W form)
    """)
    assert dz[0].startswith(tile) and dz[1:] == [grid, parts]
