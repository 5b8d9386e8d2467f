// The rules of the key exchange inside a resident group (wind_group_kernel.h), as plain functions of the iteration: the kernels go by
// them, and a host model of the exchange runs them under schedules that a GPU hardly ever shows.
#pragma once

namespace wind {

// Keys alternate between two buffers, and in bf16 groups a word's tag bit tells its iteration from the one two before it.
constexpr int group_key_buffer(int it) { return it & 1; }
constexpr int group_key_tag(int it) { return (it >> 1) & 1; }
// Keys of iteration `it` replace those of it - 2, which everybody must have read.  Where every workgroup has keys of every iteration
// that all wait for (a column part, and the row tile of all slots), a writer knows that: it holds everybody's keys of it - 1.
constexpr bool group_keys_suffice(int nparts, int column_groups, int row_groups) { return row_groups == 1 && nparts >= column_groups; }
// Else (a workgroup whose column parts are all past the vocabulary, or whose row tile has no utterance left, publishes no key that
// anybody waits for) every workgroup publishes how many iterations it has decided, and a writer waits until all have this many.
// Either way no two workgroups are more than two iterations apart, as the tag needs.
constexpr int group_keys_need(int it) { return it - 1; }

// The slots with a label (wind_group_vocab_kernel.h), as one wave of a workgroup lists them for the steps behind iteration `it - 1`: the others read the
// list until the end of iteration `it`, and that wave writes the next one as soon as it has the decisions, with no barrier in between.
constexpr int vocab_emit_list(int it) { return it & 1; }

}  // namespace wind
