"""The two counters that the waves of a slab kernel meet at: csrc/lmkan_gate.h, compiled for the host, under waves that
run in any order and at any speed, some of them without samples.  No slab is read before all of it has landed, none is
overwritten before all have read it, every walk ends, and the kernels make the calls in the order that is run here."""
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_07103_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>
#include <random>
#include <vector>
#include "lmkan_gate.h"

static const int kMost = 16, kStack = 1 << 16;
static std::mt19937 rng;
static ucontext_t scheduler, wave_context[kMost];
static std::vector<char> stacks(kMost * kStack);
static bool ended[kMost], idle[kMost];
static int now, pairs, waves, landed, read_, slab[2][kMost], on_its_way[kMost];
static bool plant;       // a mistake: waves without samples do not wait for the first slab
static const char *wrong;

static void pause()
{
    if (rng() % 3) swapcontext(&wave_context[now], &scheduler);
}

struct Counters {
    void arrive_landed() const { pause(), ++landed, pause(); }
    void arrive_read() const { pause(), ++read_, pause(); }
    void until_landed(int n) const
    {
        if (plant && idle[now] && n == waves) return;
        while (landed < n) swapcontext(&wave_context[now], &scheduler);
    }
    void until_read(int n) const
    {
        while (read_ < n) swapcontext(&wave_context[now], &scheduler);
    }
    void own_landed() const
    {
        pause();
        const int i = on_its_way[now];
        if (i >= 0) slab[i & 1][now] = i, on_its_way[now] = -1;
    }
};

// what a buffer held is gone as soon as a slab is on its way to it
static void request(int i, bool wanted)
{
    if (wanted) slab[i & 1][now] = -1, on_its_way[now] = i;
    pause();
}
static void reads(int i)
{
    for (int w = 0; w < waves; ++w)
        if (slab[i & 1][w] != i) wrong = "a slab is read that is not there";
    pause();
}

template <int WAVES>
static void walk()
{
    const lmkan::GateOrder<Counters> gate;
    if (pairs > 0) {
        request(0, true);
        gate.slab_landed();
    }
    if (idle[now]) {
        gate.feed_only<WAVES>(pairs, request);
    } else {
        for (int i = 0; i < pairs; ++i) {
            gate.wait_landed<WAVES>(i);
            reads(i);
            gate.wait_read<WAVES>(i);
            request(i + 1, i + 1 < pairs);
            reads(i);
            gate.slab_landed();
            reads(i);
            gate.slab_read();
        }
    }
    ended[now] = true;
    swapcontext(&wave_context[now], &scheduler);
}

template <int WAVES>
static const char *launch()
{
    waves = WAVES, landed = read_ = 0, wrong = nullptr;
    double weight[WAVES];
    const int without = rng() % WAVES;
    for (int w = 0; w < WAVES; ++w) {
        ended[w] = false, idle[w] = w < without, slab[0][w] = slab[1][w] = on_its_way[w] = -1;
        const double u = rng() / 4294967296.0;
        weight[w] = u * u * u + 1e-2;     // some waves hardly get a turn
        getcontext(&wave_context[w]);
        wave_context[w].uc_stack.ss_sp = &stacks[w * kStack];
        wave_context[w].uc_stack.ss_size = kStack;
        makecontext(&wave_context[w], (void (*)())walk<WAVES>, 0);
    }
    for (int turn = 0; turn < 200000; ++turn) {
        double total = 0;
        for (int w = 0; w < WAVES; ++w) total += ended[w] ? 0 : weight[w];
        double u = total * (rng() / 4294967296.0);
        const bool all = total == 0;
        for (int w = 0; w < WAVES; ++w)
            if (!ended[w]) {
                now = w;
                if ((u -= weight[w]) < 0) break;
            }
        if (all) return wrong ? wrong : landed == WAVES * pairs + (pairs > 0 ? WAVES : 0) && read_ == WAVES * pairs ? nullptr : "a count is off";
        for (int n = 1 + rng() % 20; n-- && !ended[now];) swapcontext(&scheduler, &wave_context[now]);
    }
    return "a wave waits for ever";
}

int main(int, char **argv)
{
    rng.seed(atoi(argv[1]));
    plant = atoi(argv[2]);
    for (int run = 0; run < 300; ++run) {
        pairs = rng() % 8;
        const int which = rng() % 5;
        const char *what = which == 0 ? launch<2>() : which == 1 ? launch<3>() : which == 2 ? launch<4>() : which == 3 ? launch<8>() : launch<16>();
        if (what) {
            printf("%d waves, %d pairs: %s\n", waves, pairs, what);
            return 1;
        }
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def gate(tmp_path_factory):
    folder = tmp_path_factory.mktemp("gate")
    source, program = folder / "gate.cpp", folder / "gate"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, "-o", str(program), str(source)], check=True)
    return lambda seed, plant=0: subprocess.run([str(program), str(seed), str(plant)], capture_output=True, text=True, timeout=120)


@pytest.mark.parametrize("seed", range(4))
def test_slabs_are_read_complete_and_every_walk_ends(gate, seed):
    """Zero to seven pairs, 2 to 16 waves."""
    got = gate(seed)
    assert got.returncode == 0, got.stdout


def test_the_model_sees_a_missing_wait(gate):
    """Without the wait for the first slab a wave that only fetches reports its second one too early."""
    got = gate(0, plant=1)
    assert got.returncode == 1 and "not there" in got.stdout


def test_the_kernels_make_the_calls_in_this_order():
    """Every function that has a gate, by the text of its body: the order of walk() above."""
    call = re.compile(r"gate\.(?:template )?(init|slab_landed|feed_only|wait_landed|wait_read|slab_read)\b|(__syncthreads\(\))|"
                      r"\b(?:feed\.issue|issue_piece|fill_whole)(\()")
    found = 0
    for name in ("lmkan_slab.hip", "lmkan_slab_f16.hip", "lmkan_slab_split.h"):
        with open(os.path.join(CSRC, name)) as f:
            text = re.sub(r"//[^\n]*", "", f.read())
        for body in re.split(r"\n}\n", text):
            if "SlabGate gate;" not in body:
                continue
            found += 1
            # (the part for 16-bit tables, which has a barrier per pair, and what a wave without samples requests)
            body = re.sub(r"\} else \{(?:[^{}]|\{[^{}]*(?:\{[^{}]*\}[^{}]*)*\})*\}", "}", body)
            body = re.sub(r"gate\.feed_only<.*?\n? *return;", "gate.feed_only; ", body, flags=re.S)
            calls = ["".join(m) for m in call.findall(body)]
            order = [c for c in calls if c not in ("(", "__syncthreads()")]
            assert order == ["init", "slab_landed", "feed_only", "wait_landed", "wait_read", "slab_landed", "slab_read"], (name, calls)
            at = {c: i for i, c in reversed(list(enumerate(calls)))}
            assert at["init"] < at["__syncthreads()"] < at["slab_landed"] and at["("] < at["slab_landed"], (name, calls)
            last = len(calls) - 1 - calls[::-1].index("(")          # the request of the next slab
            assert calls[last - 1] == "wait_read" and calls[last + 1] == "slab_landed", (name, calls)
    assert found == 11, found
