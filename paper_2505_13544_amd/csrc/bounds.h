// What lengths and starts out of the caller's arrays count as.  They are read on the device, where nothing can return an error
// in front of the launch, so every kernel takes them through the functions here and all of them agree.
#pragma once

namespace mtla {

// The live slots of a sequence of `len` tokens.  A length outside 0 .. max_slots * stride counts as the nearer end.
[[gnu::always_inline]] constexpr int live_slots(int len, int stride, int max_slots) {
  const int n = len > 0 ? (int)((unsigned)(len - 1) / (unsigned)stride) + 1 : 0;
  return n < max_slots ? n : max_slots;
}

// May `n` tokens be appended to a sequence of `len`?  0, or the status that refuses them (the sequence is left untouched):
// 1 (MTLA_ERR_INVALID_ARG) for a length below zero, 3 (MTLA_ERR_CAPACITY) for more than the capacity holds.
[[gnu::always_inline]] constexpr int append_status(int len, int n, int stride, int max_slots) {
  return len < 0 ? 1 : ((long long)len + n > (long long)max_slots * stride ? 3 : 0);
}

// The slots in front of a sequence's new rows.  A start outside the `past` slots that the call declared counts as all of them
// (the front launch raises the status word): no kernel leaves its arrays, and the sequence's rows are meaningless.  (As an
// unsigned number a start below zero lies above every slot that past * stride < 2^31 tokens can have.)
[[gnu::always_inline]] constexpr int slots_inside(int pos0, int stride, int past) {
  const unsigned k = (unsigned)pos0 / (unsigned)stride;
  return k < (unsigned)past ? (int)k : past;
}
// The tokens in front of them: the start itself, or those of the whole past.
[[gnu::always_inline]] constexpr int start_inside(int pos0, int stride, int past) {
  return pos0 >= 0 && (unsigned)pos0 / (unsigned)stride <= (unsigned)past ? pos0 : past * stride;
}

// The new rows of a sequence, of at most T.  A sequence's part of past + T rows then has slots_inside(..) + new_rows(..) in use.
[[gnu::always_inline]] constexpr int new_rows(int n_new, int T) { return n_new < 0 ? 0 : (n_new < T ? n_new : T); }

}  // namespace mtla
