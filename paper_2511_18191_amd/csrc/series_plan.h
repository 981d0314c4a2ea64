// Index rules of the passes that take a series per workgroup (series_f32.hip), in plain C++ so that they can be checked without a GPU
// (tests/test_series_plan.py).
#pragma once

namespace tsd {

// Where token `at` of a page starts in a layer's pool, for a model of H heads of HD and pages of PT tokens: the element of its keys of
// head 0; a head's keys are PT * HD long, the values H of those behind.  64 bits: the pool of 131072 series of 64 tokens at width 128 has
// 2^31 elements.
constexpr long kv_token(int page, int at, int H, int PT, int HD) { return (long)page * (2 * H * PT * HD) + at * HD; }

// Whether a context of so many tokens of n series is worth a workgroup per series and model, which takes it 32 tokens (or, where that
// does not fit, 16) at a time; wide: the wider model's width.
//   * A few series with a long context leave the chip idle, where the launches of the tiled path do not get longer: two blocks at width
//     64 and one at 128 pay for any number of series, each one more for 64 series more (launch by launch / this, us, one series: 2 layers of
//     64, 31 tokens 95 / 36, 63 tokens 96 / 68, 95 tokens 99 / 135; 3 layers of 128, 31 tokens 158 / 118, 63 tokens 163 / 238.  As a
//     ratio, a deep target and a one-layer draft, for which it is least: 8 layers of 64, 96 tokens 1.08 for 64 series, 128 tokens 0.75 for 64,
//     0.99 for 112 and 1.37 for 129; 8 of 128, 64 tokens 1.16 for 64, 96 tokens 0.74 for 64 (3 layers), 0.95 for 112, 1.00 for 128).
//   * A workgroup's products are 16 rows high however few its tokens are, where the tiled path fills its tiles with many series: of fewer
//     than 12 tokens only so many series (ratios at the limit, widths 32 to 128: 1 token, 512 series 1.04 to 2.4; 3 tokens, 768 1.15 to
//     1.83; 5 tokens, 1024 1.00 to 1.04 at 128; 7 tokens, 1280 1.17.  Behind it: 1 token, 768 series 0.87 at 128, 2048 0.40 to 0.78; 3
//     tokens, 2048 0.63 to 0.89; 7 tokens, 2048 0.90 to 1.10).
//   * More than 16384 series were not worth it at width 32 (16 tokens, 65536 series 1.09, 17 tokens 0.91, 12 tokens 0.84).
constexpr bool series_context_pays(int wide, int n, int tokens) {
  const int more = (tokens + 31) / 32 - (wide <= 64 ? 2 : 1);
  return tokens <= 128 && n >= 64 * more && n <= (tokens < 12 ? 128 * (tokens + 3) : 16384);
}

}  // namespace tsd
