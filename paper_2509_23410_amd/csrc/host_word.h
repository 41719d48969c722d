// A word of host memory that kernels can write, held for the length of a call: how a packing kernel reports to the host without a copy from the
// device behind it (a call of its own of about 10 us, and the wait for it).  The 64 words are one page that the first call allocates and the process
// keeps; a call that finds all of them held waits for one (each is held between a launch and the end of its stream's work, by a thread that waits for
// nothing else).
#pragma once
#include <stdint.h>

class HostWord {
public:
    HostWord();    // zero, or valid() is false: no memory
    ~HostWord();
    HostWord(const HostWord&) = delete;
    HostWord& operator=(const HostWord&) = delete;
    bool valid() const { return slot_ >= 0; }
    uint32_t* device() const;
    uint32_t value() const;

private:
    int slot_ = -1;
};
