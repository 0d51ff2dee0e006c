// Which schedule a decode step's attention takes, and the chunk of the static one: plain arithmetic, without device code, so that the
// host can hold it to the times it stands for.
#pragma once

namespace mtla {

// Slots of a chunk: about two workgroups per compute unit (256 CUs) when every sequence of the session is full; a workgroup's
// four wavefronts take 16-slot tiles round-robin, so chunks are multiples of 64 slots.
constexpr int decode_chunk(int max_batch, int max_slots) {
  const long long total = (long long)max_batch * max_slots, chunk = ((total + 511) / 512 + 63) / 64 * 64;
  return (int)(chunk < 64 ? 64 : (chunk > 1024 ? 1024 : chunk));
}

// Whether a call of `batch` sequences of up to `max_slots` slots takes the balanced schedule rather than static chunks; `chunk_set`: by the caller.
// The balanced one has a fixed cost, the scan of the lengths and a cold start of every persistent workgroup, some 5 us of a step beside a
// chunk a workgroup, and its partials are halves.  Below 8 tiles of 16 slots a unit it is left out: with partials in fp32, as the chunks' are, it would gain there only with
// two head tiles at r = 512 and some sequences (us a step, chunks / balanced, all sequences of a session, 20 and 32 heads: 24 x 1000 (1512 tiles) 31.7 / 30.4 and 35.8 / 33.9,
// 12 x 2600 33.0 / 31.0 and 38.9 / 33.4, 16 x 1024 (1024 tiles) 24.9 / 28.4 and 27.6 / 30.7; 16 heads, 24 x 1000 28.8 / 29.0; r = 256, 32 heads x 64, 24 x 1000 23.2 / 24.4),
// and the longer a softmax reference is kept, the fewer weights are exact: against 64 bits the output's error is 3.9e-4 of it in chunks and 1.10e-3 balanced
// (20 heads, 24 x 1000, queries and keys of standard deviations 2 and 1; 9.2e-4 and 1.29e-3 with queries of 1).
//
// Beyond, chunks are the faster ones at r = 128 and, with one head tile, r = 256, within three limits.
// `most`: the slots that the fullest unit has beyond its even share.  (The chunk is made for the session's sequences: a call of some of them has
// chunks as long, but fewer.)  us a step, chunks / balanced, by these slots; sequences of the call / the session x slots:
//   r = 128, 8 heads   112 / 112 x 1024 (64) 17.6 / 21.3, 24 / 128 x 2048 (320) 15.9 / 19.0, 36 / 256 x 1024 (368) 15.7 / 16.5, 112 / 224 x 1024 (448) 21.9 / 21.3,
//                      14 / 28 x 8192 (448) 21.6 / 20.6, 90 / 512 x 1024 (664) 21.1 / 20.2, 6 / 64 x 8192 (832) 19.6 / 16.6
//   r = 128, 20 heads  112 / 112 x 1024 (64) 24.2 / 30.5, 56 / 224 x 1024 (224) 20.2 / 21.8, 32 / 224 x 1024 (320) 19.2 / 18.3, 40 / 512 x 1024 (864) 27.8 / 19.5
//   r = 256, 8 heads   64 / 64 x 1024 (0) 19.6 / 22.5, 128 / 128 x 1024 (0) 25.2 / 27.1, 32 / 128 x 1024 (128) 18.8 / 18.9, 40 / 160 x 1024 (160) 20.4 / 19.5, 96 / 96 x 1024
//                      (192) 26.8 / 24.7, 24 / 128 x 2048 (320) 24.0 / 21.7, 6 / 64 x 8192 (832) 31.3 / 20.6
//   r = 256, 32 heads x 128, 32 / 32 x 1024 (0) 29.6 / 26.4; r = 512, 16 heads, 32 / 32 x 1024 (0) 31.8 / 29.1
// The chunk's length: r = 256, 8 heads, chunks of 256 (256 x 512) 25.5 / 28.2, of 384 (256 x 768) 37.3 / 32.9, of 768 52.5 / 48.3.  At r = 128 lengths that are all
// alike gain with any chunk (of 512, 24.9 / 29.0, of 1024 36.9 / 41.2), but where they range from nothing to the most, two chunks a unit: of 320 17.5 / 20.7
// (64 x 2560) and 16.5 / 19.1 (16 x 10240), of 384 21.0 / 21.1 and 21.0 / 20.0, of 1024 32.3 / 30.1 and 31.7 / 28.6.
// With two head tiles the chunks of a sequence, lengths from nothing to the most, 20 heads: two (256 x 512) 24.8 / 28.4, eight (64 x 2048) 24.1 / 23.6, 32 (16 x 8192) 26.6 / 22.9.
// A chunk that the caller set may be far from any of these: there the fixed border.
constexpr bool decode_balanced(int r, int n_heads, int batch, int max_slots, int chunk, bool chunk_set, int n_cu) {
  if (batch * ((max_slots + 15LL) / 16) < 8LL * n_cu) return false;
  const bool two = n_heads > 16;
  const int most = r == 128 ? (two ? 300 : 400) : (r == 256 && !two ? 128 : -1);
  if (chunk_set || most < 0) return true;
  const long long of_a_sequence = (max_slots + chunk - 1LL) / chunk, on_a_unit = (batch * of_a_sequence + n_cu - 1) / n_cu;
  const int longest = r == 256 ? 256 : (two || on_a_unit == 1 ? 512 : 320);
  return chunk > longest || (two && of_a_sequence > 8) || on_a_unit * chunk - (long long)batch * max_slots / n_cu > most;
}

}  // namespace mtla
