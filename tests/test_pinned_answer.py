"""The wait between a launch that writes into pinned host memory and the memory's return (csrc/pinned_answer.h), compiled for the host: the memory outlives
the writes also where the library reports an error behind the launch, or something throws before the wait."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <stdexcept>
#include "pinned_answer.h"
using namespace srigl;
// A launch writes the answer at the polls_left-th look at it; a stream is busy until then.
struct World { long polls_left; StreamState when_done; bool written = false, kept = false; long asked = 0; };
static auto answer_of(World& w) {
    return PinnedAnswer([&w] { if (w.polls_left > 0 && --w.polls_left == 0) w.written = true; return w.written; },
                        [&w] { ++w.asked; return w.polls_left > 0 ? StreamState::kBusy : w.when_done; }, [&w] { w.kept = true; });
}
#define EXPECT(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
int main() {
    {   // the usual call
        World w{1000, StreamState::kIdle};
        auto a = answer_of(w);
        EXPECT(a.launch([] { return SRIGL_OK; }) == SRIGL_OK && a.wait() && a.wait() && w.written && w.asked == 0);
    }
    for (long polls : {1L, 300000L}) {   // an error found behind the launch: the object ends only after the write
        World w{polls, StreamState::kIdle};
        { auto a = answer_of(w); EXPECT(a.launch([] { return SRIGL_ERR_HIP; }) == SRIGL_ERR_HIP); }
        EXPECT(w.written && !w.kept);
    }
    {   // an exception before the wait
        World w{200000, StreamState::kIdle};
        try {
            auto a = answer_of(w);
            a.launch([] { return SRIGL_OK; });
            throw std::runtime_error("no memory");
        } catch (const std::runtime_error&) {}
        EXPECT(w.written && !w.kept);
    }
    for (srigl_status refused : {SRIGL_ERR_INVALID_ARG, SRIGL_ERR_CAPACITY, SRIGL_ERR_UNSUPPORTED}) {   // refused before a launch: no wait
        World w{1L << 40, StreamState::kIdle};
        { auto a = answer_of(w); a.launch([&] { return refused; }); EXPECT(!a.wait()); }
        EXPECT(w.polls_left == 1L << 40 && w.asked == 0);
    }
    {   // nothing launched: no wait
        World w{1L << 40, StreamState::kIdle};
        { auto a = answer_of(w); }
        EXPECT(w.polls_left == 1L << 40);
    }
    for (StreamState s : {StreamState::kIdle, StreamState::kUnknown}) {   // a stream that ends without the answer, and one that cannot say
        World w{0, s};
        { auto a = answer_of(w); a.launch([] { return SRIGL_OK; }); EXPECT(!a.wait()); }
        EXPECT(w.asked == 1 && w.kept == (s == StreamState::kUnknown));
    }
    printf("answers ok\n");
}
"""


def test_memory_outlives_the_writes(tmp_path):
    src = tmp_path / "answers.cpp"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2305_02299_amd", "csrc"),
                    "-o", str(tmp_path / "answers"), str(src)], check=True)
    r = subprocess.run([str(tmp_path / "answers")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "answers ok" in r.stdout, (r.stdout + r.stderr)[-500:]
