// A word of host memory that kernels can write, held for the length of a call: how a packing kernel reports to the host without a copy from the
// device behind it (a call of its own of about 10 us, and the wait for it).  The words are pages of 64; a call that finds all of them held adds a
// page - it must not wait for another call's word, which is held until all work in front of it on that call's stream has ended, and that may take something
// that only the waiting call's thread does.  Pages are kept (releasing pinned memory waits for the device): as many as 64ths of the calls that ever ran at
// the same time.
#pragma once
#include <stdint.h>

struct HostWordPage;

class HostWord {
public:
    HostWord();    // zero, or valid() is false: no memory
    ~HostWord();
    HostWord(const HostWord&) = delete;
    HostWord& operator=(const HostWord&) = delete;
    bool valid() const { return page_ != nullptr; }
    uint32_t* device() const;
    uint32_t value() const;

private:
    HostWordPage* page_ = nullptr;
    int slot_ = -1;
};
