"""The words that packing kernels report in (csrc/host_word.hip), compiled for the CPU with the allocation replaced: any number of calls at once gets a word of
its own without waiting for another's, as each may wait for work that only a later call lets finish."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_23410_amd", "csrc")

PROGRAM = r"""
#include "host_word.hip"
#include <assert.h>
#include <stdlib.h>
#include <memory>
#include <set>
#include <thread>
#include <vector>

static int pages = 0;
static bool refuse = false;
extern "C" hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
    if (refuse) return hipErrorOutOfMemory;
    *p = calloc(1, bytes);
    ++pages;
    return hipSuccess;
}
extern "C" hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
extern "C" hipError_t hipHostFree(void* p) { free(p); --pages; return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }

int main() {
    refuse = true;
    { HostWord none; assert(!none.valid()); }
    refuse = false;
    for (int turn = 0; turn < 3; ++turn) {
        std::vector<std::unique_ptr<HostWord>> words;
        std::set<uint32_t*> seen;
        for (int i = 0; i < 200; ++i) {
            words.emplace_back(new HostWord);
            assert(words.back()->valid() && words.back()->value() == 0 && seen.insert(words.back()->device()).second);
            *words.back()->device() = 1000 + i;          // what a kernel writes
        }
        for (int i = 0; i < 200; ++i) assert(words[i]->value() == 1000u + i);
        for (int i = 0; i < 200; i += 3) words[i].reset();
        refuse = true;                                    // a third of them free again: no new page is asked for
        for (int i = 0; i < 200; i += 3) {
            words[i].reset(new HostWord);
            assert(words[i]->valid() && words[i]->value() == 0);
        }
        { std::vector<std::unique_ptr<HostWord>> more;    // ... and where one is and none can be had, the call is refused
          for (int i = 0; i < 64; ++i) more.emplace_back(new HostWord);
          assert(!more.back()->valid()); }
        refuse = false;
    }
    assert(pages == 4);                                    // as many as 200 at once need, kept
    std::vector<std::thread> threads;
    for (int t = 0; t < 16; ++t)
        threads.emplace_back([t] {
            for (int i = 0; i < 2000; ++i) {
                std::unique_ptr<HostWord> w[9];
                for (auto& p : w) { p.reset(new HostWord); *p->device() = (uint32_t)(9 * t + (&p - w) + 1); }
                for (auto& p : w) assert(p->value() == (uint32_t)(9 * t + (&p - w) + 1));
            }
        });
    for (auto& t : threads) t.join();
    return 0;
}
"""


def test_no_call_waits_for_a_word(tmp_path):
    (tmp_path / "words.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, "-o", str(tmp_path / "words"), str(tmp_path / "words.cpp"), "-lpthread"],
                   check=True, capture_output=True, text=True)
    subprocess.run([str(tmp_path / "words")], check=True, timeout=60)
