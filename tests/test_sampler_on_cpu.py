"""The sampler's kernel source (csrc/sampler.hip) run on the CPU, a workgroup of 1024 fibers at a time (host/simt.h): every access to LDS
is recorded, and two waves that touch a word without a barrier in between fail the test, whatever the result was.  The waves run one
after the other from barrier to barrier, in several orders, so that what no barrier orders really happens out of order.  Needs g++, no GPU."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import philox, sampler

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
MAIN = """
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "simt_run.h"
// rows vocab vec top_p inv_t key_add seed step eos bias order, then the logits on stdin: token and log-probability of each row
int main(int, char **a) {
    const int rows = atoi(a[1]), vocab = atoi(a[2]), vec = atoi(a[3]), step = atoi(a[8]), eos = atoi(a[9]), order = atoi(a[11]);
    const float top_p = strtof(a[4], 0), inv_t = strtof(a[5], 0), key_add = strtof(a[6], 0), bias = strtof(a[10], 0);
    const uint64_t seed = strtoull(a[7], 0, 10);
    std::vector<float> x((size_t)rows * vocab + 4), lp(rows);
    float *logits = (float *)(((uintptr_t)x.data() + 15) / 16 * 16);
    if (fread(logits, 4, (size_t)rows * vocab, stdin) != (size_t)rows * vocab) return 2;
    std::vector<uint64_t> uid(rows);
    std::vector<int32_t> tok(rows);
    for (int r = 0; r < rows; ++r) {
        uid[r] = r + 51;
        blockIdx.x = r;
        auto go = [&](auto kernel) { kernel(logits, nullptr, vocab, inv_t, top_p, key_add, seed, uid.data(), nullptr, step, eos, bias, tok.data(),
                                            lp.data(), nullptr, nullptr, nullptr, nullptr); };
        std::string seen;
        const int bad = simt_run(1024, order, [&]() {
            if (top_p < 1.0f) vec == 4 ? go(pc::sample_kernel<4, true, false>) : go(pc::sample_kernel<1, true, false>);
            else vec == 4 ? go(pc::sample_kernel<4, false, false>) : go(pc::sample_kernel<1, false, true>);
        }, &seen);
        if (bad) {
            printf("row %d: %s\\n", r, seen.c_str());
            return 1;
        }
        printf("%d %a\\n", tok[r], (double)lp[r]);
    }
    fprintf(stderr, "%ld tokens put in bins\\n", simt_word_adds);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    d = str(tmp_path_factory.mktemp("simt"))
    text = open(os.path.join(ROOT, "paper_2605_26606_amd", "csrc", "sampler.hip")).read()
    text = text[:text.index("void launch_sample(")].replace('#include "pc_internal.h"', '#include "simt.h"') + "}   // namespace pc\n" + MAIN
    src = os.path.join(d, "sampler.cpp")
    with open(src, "w") as f:
        f.write(text)
    common = [gxx, "-std=c++17", "-I", HOST, "-Wno-unknown-pragmas", "-Wno-psabi"]
    # (no contraction of products and sums: what the source does not say with fmaf is two roundings here)
    for cmd in (common + ["-O1", "-ffp-contract=off", "-fsanitize=thread", "--param", "tsan-instrument-func-entry-exit=0", "-c", src, "-o", src + ".o"],
                common + ["-O2", "-c", os.path.join(HOST, "simt.cpp"), "-o", os.path.join(d, "simt.o")],
                [gxx, src + ".o", os.path.join(d, "simt.o"), "-o", os.path.join(d, "run")]):
        p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert p.returncode == 0, p.stdout[-4000:]
    return os.path.join(d, "run")


def _run(program, x, T, top_p, seed, step, eos, bias, order, said=None):
    n, V = x.shape
    inv_t = np.float32(1.0) / np.float32(T)
    key_add = np.float32(bias) * np.float32(T) if eos >= 0 else np.float32(0)
    args = [n, V, 4 if V % 4 == 0 else 1, float(np.float32(top_p)), float(inv_t), float(key_add), seed, step, eos, bias, order]
    p = subprocess.run([program] + [repr(a) for a in args], input=np.ascontiguousarray(x, dtype=np.float32).tobytes(), stdout=subprocess.PIPE,
                       stderr=subprocess.PIPE, timeout=300)
    out = p.stdout.decode()
    assert p.returncode == 0, "%s%s" % (out[-500:], p.stderr.decode()[-500:])
    lines = [l.split() for l in out.splitlines()]
    if said is not None:
        said.append(p.stderr.decode())
    return [int(t) for t, _ in lines], [float.fromhex(lp) for _, lp in lines]


def _rows(form, V, rng, n=2):
    x = rng.standard_normal((n, V)).astype(np.float32)
    if form == "late":       # masked beginnings of every wave's segment: the bins' ring goes round
        seg = -(-(-(-V // 16)) // 256) * 256
        x[:, np.arange(V) % seg < seg // 2] = -1e9
    elif form == "outlier":  # one token far above all that is seen of the row at first
        x[:, V - 3] += 150.0
    elif form == "ties":     # few different logits: the cut falls among ties, in the list or (rows of one value) beyond it
        x = np.round(x * 2) / 2 + 0.0   # (no negative zeros: the keys order those behind the others)
        x[1] = 0.5
    elif form == "close":    # all in one bin: it is cut into parts, and the part with the cut, of several tokens, once more
        x = np.float32(1) + np.float32(2.0 ** -22) * rng.integers(0, 8000, (n, V)).astype(np.float32)
    elif form == "peaked":
        x[:, 3::97] += 9.0
    return x.astype(np.float32)


@pytest.mark.parametrize("order", [0, 1, 5])
@pytest.mark.parametrize("V,top_p", [(4100, 1.0), (4100, 0.9), (2051, 0.7), (6144, 0.999)])
@pytest.mark.parametrize("form", ["bulk", "peaked", "late", "outlier", "ties", "close"])
def test_no_races_between_waves_and_the_oracles_tokens(program, form, V, top_p, order):
    # (tolerances as on the GPU: the weights are float32, a uniform on the rounding of a boundary may go either way)
    rng = np.random.default_rng(V + len(form))
    x, T, eos, bias = _rows(form, V, rng), 0.9, V // 2, 0.25
    tok, lp = _run(program, x, T, top_p, 5, 1, eos, bias, order)
    for i in range(len(x)):
        u = philox.sampling_uniform(5, 51 + i, 1)
        want, wlp = sampler.sample_token(x[i] * np.float32(1.0 / np.float32(T)), 1.0, u, eos, bias, top_p=top_p)
        assert tok[i] == want and abs(lp[i] - wlp) <= 3e-5 * max(1.0, abs(wlp))


@pytest.mark.parametrize("V", [4100, 2051])
def test_one_rounding_of_the_biased_logit_on_every_way(program, V):
    # Nothing but the cut distinguishes the nucleus from plain sampling with the other tokens masked: the same bits, also where the EOS id has
    # the largest logit and is drawn.
    rng = np.random.default_rng(V)
    x = rng.standard_normal((8, V)).astype(np.float32)
    T, top_p, eos, bias = 0.7, 0.9, V // 3, 0.3
    x[:, eos] = 6.0 + rng.random(8).astype(np.float32)
    tok, lp = _run(program, x, T, top_p, 5, 2, eos, bias, 0)
    y = x.astype(np.float64) / T
    y[:, eos] += bias
    w = np.exp(y - y.max(1, keepdims=True))
    keep = np.stack([sampler.nucleus(r, top_p) for r in w])
    want = _run(program, np.where(keep, x, -np.inf).astype(np.float32), T, 1.0, 5, 2, eos, bias, 0)
    assert (tok, lp) == want and eos in tok


@pytest.mark.parametrize("V,shift", [(4100, 2.0e5), (4097, 2.0e5), (262152, 0.0), (4100, 9.9e4)])
def test_rows_beyond_the_bins_are_not_put_in_them(program, V, shift):
    # Scaled logits beyond 1e5 and rows of more than 2^18 tokens go to the other search whatever the bins hold.
    rng = np.random.default_rng(V)
    x = (rng.standard_normal((1, V)) + shift).astype(np.float32)
    said = []
    tok, lp = _run(program, x, 1.0, 0.9, 5, 1, V // 2, 0.25, 0, said)
    want, wlp = sampler.sample_token(x[0], 1.0, philox.sampling_uniform(5, 51, 1), V // 2, 0.25, top_p=0.9)
    assert tok[0] == want and abs(lp[0] - wlp) <= 3e-5 * max(1.0, abs(wlp))
    assert said[0].startswith("0 tokens") == (shift > 1e5 or V > 1 << 18)
