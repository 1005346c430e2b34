// A call made without the interpreter's lock.  CPython only.
#pragma once

#include <Python.h>

#include <utility>

namespace swimba {

// f() with the lock released; it is held again when the call returns and when it throws, so that whoever
// catches may set a Python exception.
template <typename F>
auto unlocked(F &&f)
{
    struct Released {
        PyThreadState *state = PyEval_SaveThread();
        ~Released() { PyEval_RestoreThread(state); }
    } released;
    return std::forward<F>(f)();
}

}  // namespace swimba
