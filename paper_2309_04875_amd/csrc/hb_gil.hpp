// The interpreter lock around a call of the C ABI from the Python binding.
#pragma once

#include <Python.h>

// Gives the lock up for its lifetime: taken again on every way out of the scope, that of an exception among them, for whoever
// catches it goes on with Python objects.
class WithoutGil {
  public:
    WithoutGil() : state_(PyEval_SaveThread()) {}
    ~WithoutGil() { PyEval_RestoreThread(state_); }
    WithoutGil(const WithoutGil &) = delete;
    WithoutGil &operator=(const WithoutGil &) = delete;

  private:
    PyThreadState *state_;
};

template <class Call>
int without_gil(const Call &call)
{
    const WithoutGil released;
    return call();
}
