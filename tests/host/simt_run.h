#pragma once
#include <functional>
#include <string>
// One workgroup of `threads` threads.  order 0: the waves in order between two barriers, 1: the last one first, more: mixed.  0 if no race was
// seen and every barrier was met by all waves; else 1 and what was seen.
int simt_run(int threads, int order, const std::function<void()> &kernel, std::string *report);
