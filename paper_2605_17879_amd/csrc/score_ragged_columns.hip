// The scoring kernel for rank counts that fill no tiling exactly: the per-column route of short batches.
#define GD_SCORE_RAGGED 3
#include "score.hip"
