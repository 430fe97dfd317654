"""The rules that choose a kernel or cut its work from a call's sizes, over the whole range
that the entry points accept (no GPU needed): the rules are plain C++, compiled here with
the undefined-behaviour checks on, and compared with the same rules on Python's integers."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
INT32_MAX = 2 ** 31 - 1


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """Evaluates expressions of the rules: rules(["lanes_fit(16, 4)", ...]) -> list of int."""
    def run(exprs):
        d = tmp_path_factory.mktemp("rules")
        body = "".join(f"  std::printf(\"%lld\\n\", (long long)({e}));\n" for e in exprs)
        (d / "r.cpp").write_text('#include <cstdio>\n#include "launch_rules.hpp"\nusing namespace sdmm;\n'
                                 "int main(int argc, char**) {\n  volatile int one = argc;  // not known to the compiler\n"
                                 "  const int v = one;\n  (void)v;\n" + body + "  return 0;\n}\n")
        subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I",
                        os.path.join(ROOT, "paper_2111_13094_amd", "csrc"), str(d / "r.cpp"), "-o", str(d / "r")],
                       check=True)
        out = subprocess.run([str(d / "r")], check=True, capture_output=True, text=True).stdout
        return [int(x) for x in out.split()]
    return run


def test_draws_of_a_pass_fit_its_lanes(rules):
    """One draw per lane is chosen exactly when the S queries' draws fit 64 lanes, also where
    S * ns leaves 32 bits; and a pass of several rounds never has more than 64 draws."""
    cases = [(S, ns) for S in (1, 2, 4, 8, 16)
             for ns in (1, 2, 3, 4, 5, 15, 16, 17, 63, 64, 65, 1 << 27, (1 << 27) + 1, 1 << 28, 1 << 29, 1 << 30,
                        INT32_MAX)]
    got = rules([f"lanes_fit({S}, v * {ns})" for S, ns in cases])
    assert got == [int(S * ns <= 64) for S, ns in cases]
    fit = [(S, ns, nq) for S, ns in cases if S * ns <= 64 for nq in (1, 65535, 65536, 262144, 1 << 40)]
    for S, ns, nq, a, b in zip(*zip(*fit), rules([f"lanes_rounds({nq}LL, {S}, v * {ns})" for S, ns, nq in fit]),
                               rules([f"rounds_per_pass({S}, v * {ns}, 2)" for S, ns, nq in fit])):
        assert 1 <= a <= 4 and S * ns * a <= 64 and (a == 1 or nq >= 4096 * S * a), (S, ns, nq)
        assert b == min(2, 64 // (S * ns)), (S, ns)


def test_one_separate_draw_keeps_the_group_kernel(rules):
    """Separate draws take the lanes kernel from two draws up, while they fit the lanes and
    the table fits one L2."""
    cases = [(S, ns, t) for S in (1, 4, 16) for ns in (1, 2, 4, 64 // S, 64 // S + 1, INT32_MAX)
             for t in (128, 4 << 20, (4 << 20) + 128, 1 << 40)]
    got = rules([f"sample_by_lanes({S}, v * {ns}, {t}LL)" for S, ns, t in cases])
    assert got == [int(2 <= ns and S * ns <= 64 and t <= 4 << 20) for S, ns, t in cases]


def test_rounds_of_the_separate_calls(rules):
    """Four rounds per pass from 16384 wave groups of that many on; the pdf of groups of 4
    lanes takes one."""
    cases = [(S, n) for S in (1, 2, 4, 8, 16) for n in (1, 65535 * S, 65536 * S - 1, 65536 * S, 1 << 50)]
    got = rules([f"condition_in_rounds({S}, v * {n}LL)" for S, n in cases])
    assert got == [int(n >= 65536 * S) for S, n in cases]
    got = rules([f"pdf_in_rounds({S}, v * {n}LL)" for S, n in cases])
    assert got == [int(S <= 8 and n >= 65536 * S) for S, n in cases]


def test_staged_product_pdfs(rules):
    """The product pdf stages from 262144 queries on (400000 of more than 32 components), never
    for groups of fewer than 16 component lanes."""
    cases = [(G, nq) for G in (4, 8, 16, 32, 64) for nq in (1, 131072, 262143, 262144, 399999, 400000, 1 << 40)]
    got = rules([f"staged_pdf({G}, v * {nq}LL)" for G, nq in cases])
    assert got == [int(G >= 16 and nq >= (400000 if G == 64 else 262144)) for G, nq in cases]


def test_batches_cover_every_draw(rules):
    """The batches of G draws cover all ns draws and their first draw's index stays in 32
    bits, up to the largest ns."""
    cases = [(G, ns) for G in (4, 8, 16, 32, 64)
             for ns in (1, G - 1, G, G + 1, 1000, INT32_MAX - G, INT32_MAX - 1, INT32_MAX)]
    for (G, ns), n in zip(cases, rules([f"draw_batches(v * {ns}, {G})" for G, ns in cases])):
        assert (n - 1) * G < ns <= n * G, (G, ns)


def test_chunks_of_a_leaf_cover_it_once(rules):
    """A leaf's chunks of at most 4096 records follow each other, cover all its records and
    hold at most 4096 each, up to the largest leaf that a refinement accepts."""
    most = 4096
    counts = [1, 63, 64, 4095, 4096, 4097, 8192, 8193, 200003, 16616003, INT32_MAX - most, INT32_MAX - most + 1,
              INT32_MAX - 1, INT32_MAX]
    n_chunks = rules([f"chunks_of(v * {c}, {most})" for c in counts])
    assert n_chunks == [-(-c // most) for c in counts]
    pick = [(c, n, q) for c, n in zip(counts, n_chunks) for q in sorted({0, 1, n // 2, n - 2, n - 1}) if 0 <= q < n]
    begin = rules([f"chunk_begin(v * {c}, {n}, {q})" for c, n, q in pick])
    end = rules([f"chunk_end(v * {c}, {n}, {q})" for c, n, q in pick])
    for (c, n, q), lo, hi in zip(pick, begin, end):
        size = (-(-c // n) + 63) // 64 * 64
        assert (lo, hi) == (min(c, q * size), min(c, (q + 1) * size)) and hi - lo <= most, (c, n, q)
        assert (q > 0 or lo == 0) and (q < n - 1 or hi == c), (c, n, q)


@pytest.mark.parametrize("K,ns", [(4, 1 << 28), (16, 1 << 30), (4, 1 << 27)])
def test_calls_with_many_draws_reach_the_launch(K, ns):
    """Draw counts whose product with the queries of a wave leaves 32 bits: with no device in
    sight each call gets as far as the launch and returns its error (a wrapped product of 0
    ended the process in a division)."""
    code = ("import ctypes as C\nfrom paper_2111_13094_amd import sdmm\nL, p = sdmm.lib(), C.c_void_p(256)\n"
            f"K, ns = {K}, {ns}\n"
            "print(L.sdmm_sample(p, 1, K, p, 1, p, p, ns, None, 0, p, p, p, None, None),\n"
            "      L.sdmm_condition_sample_pdf(p, 1, K, p, p, 1, ns, None, 0, p, p, p, None),\n"
            "      L.sdmm_product_sample(p, 1, K, p, p, p, 1, K, p, p, p, 1, ns, None, 0, p, p, p, None, None))\n")
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=env, capture_output=True, text=True)
    assert r.returncode == 0, r
    assert r.stdout.split() == ["-2"] * 3
