"""The library's host side (planner, argument and call-order checks, tree tables, the per-level tables of a
drafting call, the verification-free step helpers) under AddressSanitizer and UndefinedBehaviorSanitizer on
the CPU: tests/host_fuzz.cpp replaces the HIP runtime and every kernel launcher by host stand-ins and drives
the complete call sequences with random valid and invalid inputs."""
import os
import shutil
import subprocess

import pytest

import test_gpu_few_pairs
import test_gpu_shared_tiles

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def build_and_run(tmp_path_factory, sanitize):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path_factory.mktemp("host") / "host_fuzz")
    cmd = [gxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2511_13587_amd", "csrc"), *sanitize, "-g", "-O1", "-w", "-pthread",
           os.path.join(ROOT, "paper_2511_13587_amd", "csrc", "vvs_host.cpp"), os.path.join(ROOT, "tests", "host_fuzz.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    if r.returncode != 0 and "san" in r.stderr.lower() and "cannot find" in r.stderr.lower():
        pytest.skip("the sanitizer runtime is not installed")
    assert r.returncode == 0, r.stderr[-3000:]
    env = dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0:detect_leaks=1", UBSAN_OPTIONS="print_stacktrace=1")
    return lambda *args, **kw: subprocess.run([exe, *args], capture_output=True, text=True, timeout=300, env=env, **kw)


@pytest.fixture(scope="module")
def host_fuzz(tmp_path_factory):
    return build_and_run(tmp_path_factory, ["-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-static-libasan"])


def test_contexts_on_threads_of_their_own_share_nothing_unguarded(tmp_path_factory):
    r = build_and_run(tmp_path_factory, ["-fsanitize=thread"])("threads")
    assert r.returncode == 0 and "threads ok" in r.stdout, (r.stdout[-2000:], r.stderr[-3000:])


def test_host_side_is_clean_under_sanitizers(host_fuzz):
    r = host_fuzz()
    assert r.returncode == 0 and "host fuzz ok" in r.stdout, (r.stdout[-2000:], r.stderr[-3000:])


def test_gpu_tests_reach_the_tiles_they_name(host_fuzz):
    want = [(f"partial {n} {k} {m}", (*tile, 1)) for m, n, k, tile in test_gpu_shared_tiles.PRODUCTS]
    for d, _, d_ff, tokens, qkv, gate_up in test_gpu_shared_tiles.EPILOGUES:
        want += [(f"qkv {d} {d_ff} {2 * tokens}", (*qkv, 1, 1)), (f"gate_up {d} {d_ff} {2 * tokens}", (*gate_up, 1, int(gate_up[1] >= 128)))]
    want += [(f"qkv {d} {d_ff} {2 * prompts * tokens}", (32, 32, 1, 0)) for d, _, d_ff, prompts, tokens, _ in test_gpu_few_pairs.SMALL_TILES]
    want += [("qkv 512 1408 140", (32, 32, 1, 0))]
    want += [(f"gate_up {d} {d_ff} {2 * tokens}", (*plan, 0)) for d, _, d_ff, tokens, plan in test_gpu_shared_tiles.OWN_GATE_UP]
    # ... and where gate/up shares its operands: more than one round of 32 x 64 tiles, four rounds, and more than one of 64 x 64
    want += [("gate_up 2048 8256 32", (64, 128, 1, 1)), ("gate_up 2048 32768 32", (64, 128, 1, 1)), ("gate_up 4096 8256 64", (64, 128, 1, 1))]
    r = host_fuzz("plans", input="\n".join(line for line, _ in want))
    assert r.returncode == 0, r.stderr[-3000:]
    got = [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()]
    assert len(got) == len(want)
    wrong = [(line, plan, tile) for (line, tile), plan in zip(want, got) if plan != tile]
    assert not wrong, wrong
