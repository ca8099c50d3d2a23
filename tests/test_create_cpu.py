"""The library's host side against a stand-in for the HIP runtime (create_check.cpp): what ds_create leaves
behind, and what is launched for a shape, checked without a GPU."""
import os
import re
import shutil
import subprocess

import pytest

import held_shapes as H

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_1905_05957_amd")
SIGN, TOPK, QSGD, CLIP, TERNARY = 1, 2, 3, 4, 6
RMS, NOFB_SID = 4, 8 | 16


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    binary = str(tmp_path_factory.mktemp("create") / "create_check")
    # -rdynamic: the program's own functions answer for the runtime's
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", os.path.join(HERE, "create_check.cpp"), "-o", binary,
                    "-rdynamic", "-L" + PKG, "-lds_hip", "-Wl,--unresolved-symbols=ignore-in-shared-libs",
                    f"-Wl,-rpath,{PKG}:{rocm}/lib"], check=True)
    return binary


def test_create_against_a_stand_in_runtime(program):
    r = subprocess.run([program], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "FAILED" not in r.stdout and "ok: ternary" in r.stdout, r.stdout + r.stderr


def _launches(program, calls):
    """Per call the list of (kernel, grid x, grid y)."""
    text = "".join(" ".join(str(v) for v in c) + "\n" for c in calls)
    r = subprocess.run([program, "launches"], input=text, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "failed" not in r.stdout, r.stdout + r.stderr
    out = [[(n, int(x), int(y)) for n, x, y in (line.split() for line in block.splitlines())] for block in r.stdout.split("\n.\n")[:-1]]
    assert len(out) == len(calls)
    return out


def _check(launched, kernel, tiles, workgroups, rows, shape):
    first, x, y = launched[0]
    if tiles == 0:
        assert not any("_held" in n for n, _, _ in launched) and (x, y) == (workgroups, rows), (shape, launched)
        return
    r, l = H.REGISTERS_AND_LDS[tiles]
    assert kernel in first and re.search(f"Li{r}ELi{l}EEEv", first) and (x, y) == (workgroups, rows), (shape, launched)
    # a row that one workgroup holds, and rows of up to 32 tiles in sizes of one and two, need no finish launch
    alone = workgroups == 1 or (tiles <= 2 and -(-shape[1] // 2048) <= 32)
    assert len(launched) == (1 if alone else 2), (shape, launched)
    if not alone:
        assert "_held_finish" in launched[1][0] and launched[1][1:] == (workgroups, rows), (shape, launched)


def test_worker_shapes_are_launched_as_listed(program):
    calls = [("w", SIGN, n, d, int(dtype == "bf16"), RMS * rms) for n, d, dtype, rms, _, _ in H.SIGN_WORKER]
    for shape, launched in zip(H.SIGN_WORKER, _launches(program, calls)):
        n, d, dtype, rms, tiles, workgroups = shape
        kernel = "k_sign_held_worker" + f"ILb{int(dtype == 'bf16')}ELb{int(rms)}E"
        _check(launched, kernel, tiles, workgroups, n, shape)


def test_server_shapes_are_launched_as_listed(program):
    calls = [("s", SIGN, n, d, 0, RMS * rms) for n, d, _, rms, _, _ in H.SIGN_SERVER]
    for shape, launched in zip(H.SIGN_SERVER, _launches(program, calls)):
        n, d, _, rms, tiles, workgroups = shape
        _check(launched, f"k_sign_held_serverILb{int(rms)}E", tiles, workgroups, 1, shape)


def test_ternary_shapes_are_launched_as_listed(program):
    calls = [("w", TERNARY, n, d, int(dtype == "bf16"), NOFB_SID) for n, d, dtype, _, _ in H.TERNARY]
    for shape, launched in zip(H.TERNARY, _launches(program, calls)):
        n, d, dtype, tiles, workgroups = shape
        _check(launched, f"k_tern_heldILb{int(dtype == 'bf16')}E", tiles, workgroups, n, shape)


def test_every_size_is_listed(program):
    """Several workgroups of every size, one workgroup of every size that is left to one, and separate launches stand in
    the lists; those of the ternary compressor, whose tests compare with the oracle, for one row and several of both types."""
    assert {t for *_, t, w in H.SIGN_WORKER if w > 1} == {0, 1, 2, 4, 8, 14, 24}
    assert {t for *_, t, w in H.SIGN_SERVER if w > 1} == {0, 1, 2, 4, 8, 14, 24}
    assert {t for *_, t, w in H.TERNARY if w > 1} == {0, 1, 2, 4, 8, 14, 24}
    assert {t for *_, t, w in H.SIGN_WORKER if w == 1} == {1, 2, 4, 8, 14}
    assert {t for *_, t, w in H.SIGN_SERVER if w == 1} == {1, 2, 4}
    assert {t for *_, t, w in H.TERNARY if w == 1} == {1, 2, 4}
    assert {(n > 1, dtype) for n, _, dtype, t, _ in H.TERNARY if t == 0} == {(False, "f32"), (True, "f32"), (False, "bf16"), (True, "bf16")}


@pytest.mark.parametrize("n,d,k,one", [
    (1, 65_536, 1, True), (16, 65_536, 6553, True), (16, 1000, 1, True), (64, 1000, 1, True), (64, 65_536, 1, False), (64, 40_000, 400, True),
    (64, 65_536, 6553, False), (256, 4096, 4, False), (256, 16_000, 16, False), (256, 16_000, 160, True), (256, 16_000, 1600, True),
    (1024, 1000, 1, False), (1024, 1000, 100, True), (1024, 60_040, 600, False), (1024, 65_536, 6553, False), (4096, 16_000, 16, False),
    (4096, 16_000, 1600, True), (8, 65_537, 655, False)])
def test_short_topk_rows_of_many_workers(program, n, d, k, one):
    """The worker block of a short row is one launch whatever the number of workers; the server's is where that is the
    faster way, and keeps to the launches of long rows where many messages hold few entries, or very many."""
    worker, server = _launches(program, [("w", TOPK, n, d, 0, 0, k), ("s", TOPK, n, d, 0, 0, k)])
    short = [name for name, _, _ in worker if "k_topk_slices" in name or "k_topk_solo" in name]
    assert len(short) == (len(worker) if d <= 65_536 else 0), worker
    kernels = [name for name, _, _ in server if "k_topk_dense_apply" not in name]       # that one is the update
    if one:
        assert len(kernels) == 1 and ("k_topk_slices" in kernels[0] or "k_topk_solo" in kernels[0]), server
    else:
        assert "k_topk_sub_starts" in kernels[0] and not any("k_topk_slices" in name or "k_topk_solo" in name for name in kernels), server


# the server call that the program makes has a momentum buffer
@pytest.mark.parametrize("n,d,exchange", [
    (1, 20_001, True), (8, 512 * 2048, True), (8, 512 * 2048 + 1, False), (16, 1_000_003, True), (16, 2_000_001, False), (32, 1_000_003, True),
    (32, 2_000_001, False), (33, 2_000_001, True), (48, 1280 * 2048, True), (64, 1280 * 2048 + 1, False),
    (16, 25_557_032, False)])
def test_quantiser_servers_take_the_way_that_is_faster(program, n, d, exchange):
    launched, = _launches(program, [("s", QSGD, n, d, 0, 0)])
    (name, x, y), = launched
    assert f"k_qsgd_serverILi2ELb0ELb{int(exchange)}E" in name and (x, y) == (-(-d // 2048), 1), launched


@pytest.mark.parametrize("n,d,exchange", [(8, 512 * 2048 + 1, False), (9, 768 * 2048, True), (12, 768 * 2048 + 1, False), (13, 1280 * 2048, True),
                                          (32, 1280 * 2048 + 1, False), (33, 25_557_032, True)])
def test_quantiser_servers_without_momentum_take_the_way_that_is_faster(program, n, d, exchange):
    launched, = _launches(program, [("p", QSGD, n, d, 0, 0)])
    (name, x, y), = launched
    assert f"k_qsgd_serverILi1ELb0ELb{int(exchange)}E" in name and (x, y) == (-(-d // 2048), 1), launched


@pytest.mark.parametrize("n,d,one", [(24, 4_166_667, True), (24, 4_166_666, False), (23, 25_557_032, False), (64, 1_600_000, True), (64, 1_000_003, False)])
def test_clipping_servers_take_many_long_messages_one_by_one(program, n, d, one):
    """With the update.  The program clears 15 bits: four bytes an element."""
    for block, upd in (("s", 2), ("p", 1)):
        launched, = _launches(program, [(block, CLIP, n, d, 0, 0)])
        (name, _, _), = launched
        assert f"k_clip_serverILi4ELi{upd}ELb{int(one)}E" in name, launched
