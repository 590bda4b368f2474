#pragma once
// How many words a shared buffer holds, the same value in every thread of the block.  Between two calls any thread may add to
// the buffer; `sync` is the block's barrier.  `more`: words are added again before the block's next barrier.  Then nobody may go on
// until everybody has read: a thread that leaves the first barrier late would otherwise count words of the next step, and what
// hangs on the count (a restore point, a branch with barriers in it) would differ between threads.  Plain C++ on the host, so
// that the order of its steps can be tested with threads held back there.
template <class Count, class Sync>
#if defined(__HIPCC__)
__host__ __device__
#endif
inline unsigned fill_level(const Count &count, bool more, const Sync &sync) {
    sync();
    const unsigned n = count();
    if (more) sync();
    return n;
}
