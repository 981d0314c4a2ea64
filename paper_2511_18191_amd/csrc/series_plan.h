// Index rules of the passes that take a series per workgroup (series_f32.hip), in plain C++ so that they can be checked without a GPU
// (tests/test_series_plan.py).
#pragma once

namespace tsd {

// Where token `at` of a page starts in a layer's pool, for a model of H heads of HD and pages of PT tokens: the element of its keys of
// head 0; a head's keys are PT * HD long, the values H of those behind.  64 bits: the pool of 131072 series of 64 tokens at width 128 has
// 2^31 elements.
constexpr long kv_token(int page, int at, int H, int PT, int HD) { return (long)page * (2 * H * PT * HD) + at * HD; }

}  // namespace tsd
