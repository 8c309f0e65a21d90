"""The rules by which workgroups that extract may wait for workgroups that detect (csrc/cb_claim.h), compiled for the host and run with threads as workgroups
on a limited number of places, in any order of dispatch: no launch may get stuck, every block is detected once, and every frame ends once."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1808_05488_amd", "csrc")

SOURCE = r"""
#include "cb_claim.h"
#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <mutex>
#include <random>
#include <thread>
#include <vector>

namespace {
struct Mem {
    unsigned exchange(std::atomic<unsigned>* p, unsigned v) const { return p->exchange(v); }
    int add(std::atomic<int>* p, int v) const { return p->fetch_add(v); }
};
struct Stuck {};
// a layer's device memory
struct Layer {
    std::vector<std::atomic<unsigned>> claims, mail, counts;
    std::vector<std::atomic<int>> detected;
    std::atomic<int> begun{0}, done{0}, frame{0}, ended{0}, early{0};
    Layer(int n, int e) : claims(cb::claim_words(n)), mail(n), counts(e), detected(n) {}
};
struct Chip {
    std::mutex m;
    std::condition_variable cv;
    int places;
    std::atomic<bool> stop{false};
    void enter() { std::unique_lock<std::mutex> l(m); cv.wait(l, [&] { return places > 0 || stop; }); if (stop) throw Stuck(); --places; }
    void leave() { { std::lock_guard<std::mutex> l(m); ++places; } cv.notify_all(); }
};
// in_order: extracting workgroups have the numbers in which they begin
void workgroup(Layer& L, Chip& chip, int number, int blocks, int extracting, int patience, bool in_order)
{
    Mem mem;
    std::this_thread::yield();
    const unsigned tag = (unsigned)L.frame.load() + 1u;
    auto claim = [&](int b) { return &L.claims[cb::claim_index(b, blocks)]; };
    auto end = [&]() { L.done = 0; L.begun = 0; ++L.ended; ++L.frame; };
    auto work = [&](int b) { std::this_thread::yield(); ++L.detected[b]; L.mail[b] = tag; };
    const int bid = number < blocks ? -1 : in_order ? cb::extraction_number(mem, &L.begun) : number - blocks;
    cb::detect_or_extract(
        bid >= 0,
        [&]() {
            if (cb::claim_block(mem, claim(number), tag, &L.done, false) != tag) work(number);
            else if (cb::claim_lost(mem, &L.done, extracting)) end();
        },
        [&](bool limited) {
            for (int polls = 0;; ++polls) {
                bool all = true;
                for (auto& m : L.mail) all = all && m == tag;
                if (all) return true;
                if (limited && patience >= 0 && polls >= patience) return false;
                if (chip.stop) throw Stuck();
                std::this_thread::yield();
            }
        },
        [&]() { for (int b = 0; b < blocks; ++b) if (*claim(b) != tag) return b; return -1; },
        [&](int b) {
            if (cb::claim_block(mem, claim(b), tag, &L.done, true) != tag) work(b);
            else if (cb::claim_lost(mem, &L.done, extracting)) ++L.early;       // an extracting workgroup that is not through cannot end the frame
        },
        [&]() {
            L.counts[bid] = tag;
            for (int b = 0; b < bid; ++b)
                while (L.counts[b] != tag) {
                    if (chip.stop) throw Stuck();
                    std::this_thread::yield();
                }
            if (cb::extraction_done(mem, &L.done, extracting)) end();
        });
}
}  // namespace

// order: 0 as numbered, 1 extracting workgroups first, 2 any.  Launches (one a layer) of all streams share the places.  0, or what went wrong
extern "C" int play(int places, int streams, int blocks, int extracting, int frames, int patience, int order, int in_order, int seed, int seconds)
{
    std::mt19937 rng(seed);
    Chip chip;
    chip.places = places;
    std::vector<Layer*> layers;
    for (int s = 0; s < streams; ++s) layers.push_back(new Layer(blocks, extracting));
    int wrong = 0;
    for (int f = 0; f < frames && !wrong; ++f) {
        std::vector<std::pair<int, int>> wg;
        for (int n = 0; n < blocks + extracting; ++n)
            for (int s = 0; s < streams; ++s) wg.push_back({s, order == 1 ? blocks + extracting - 1 - n : n});
        if (order == 2) std::shuffle(wg.begin(), wg.end(), rng);
        std::atomic<int> left{(int)wg.size()}, stuck{0};
        std::thread dispatch([&] {
            std::vector<std::thread> t;
            try {
                for (auto& w : wg) {
                    chip.enter();
                    t.emplace_back([&chip, &left, &stuck, &layers, w, blocks, extracting, patience, in_order] {
                        try { workgroup(*layers[w.first], chip, w.second, blocks, extracting, patience, in_order); } catch (Stuck&) { ++stuck; }
                        chip.leave();
                        --left;
                    });
                }
            } catch (Stuck&) { ++stuck; }
            for (auto& x : t) x.join();
        });
        const auto until = std::chrono::steady_clock::now() + std::chrono::seconds(seconds);
        while (left && std::chrono::steady_clock::now() < until) std::this_thread::sleep_for(std::chrono::microseconds(200));
        if (left) { std::lock_guard<std::mutex> l(chip.m); chip.stop = true; }
        chip.cv.notify_all();
        dispatch.join();
        if (stuck) wrong |= 1;
        for (auto* L : layers) {
            for (auto& d : L->detected) if (d != f + 1) wrong |= 2;
            if (L->frame != f + 1 || L->ended != f + 1 || L->done != 0) wrong |= 4;
            if (L->early) wrong |= 8;
        }
    }
    for (auto* L : layers) delete L;
    return wrong;
}
// whether n blocks have words of their own, those of 32 neighbours on different lines of 128 bytes
extern "C" int words(unsigned n)
{
    std::vector<char> seen(cb::claim_words(n));
    for (unsigned b = 0; b < n; ++b) {
        const unsigned i = cb::claim_index(b, n);
        if (i >= seen.size() || seen[i]++) return 0;
        if (b && i / 32 == cb::claim_index(b - 1, n) / 32) return 0;
    }
    return 1;
}
"""


@pytest.fixture(scope="module")
def claims(tmp_path_factory):
    d = tmp_path_factory.mktemp("claims")
    src, lib = d / "claims.cpp", d / "libclaims.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    return C.CDLL(str(lib))


@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("places,streams,blocks,extracting", [(1, 1, 9, 3), (2, 1, 30, 5), (3, 1, 8, 20), (4, 2, 12, 4), (8, 3, 20, 8), (64, 2, 24, 6)])
def test_no_launch_gets_stuck(claims, places, streams, blocks, extracting, order):
    for seed in range(4):
        for patience in (0, 1, 50):
            assert claims.play(places, streams, blocks, extracting, 4, patience, order, 1, seed, 60) == 0, (seed, patience)


@pytest.mark.parametrize("places,streams,blocks,extracting", [(4, 1, 9, 4), (8, 2, 20, 6)])
def test_the_play_sees_workgroups_that_only_wait(claims, places, streams, blocks, extracting):
    """Without an end to its patience a workgroup waits for others that never get a place."""
    assert claims.play(places, streams, blocks, extracting, 1, -1, 1, 1, 0, 1) & 1


def test_the_play_sees_workgroups_that_wait_for_later_ones(claims):
    """Numbered otherwise than they begin, extracting workgroups wait for counts that nobody publishes."""
    assert claims.play(1, 1, 9, 3, 1, 0, 1, 0, 0, 1) & 1


def test_every_block_has_a_word_of_its_own(claims):
    for n in [*range(1, 200), 1023, 1024, 1025, 2048, 4800, 32400, 524288]:
        assert claims.words(n) == 1, n
