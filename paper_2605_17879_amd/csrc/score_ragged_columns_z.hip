// The scoring kernel for rank counts that fill no tiling exactly: the per-column route of short batches, with the z output.
#define GD_SCORE_WANT_Z 1
#define GD_SCORE_RAGGED 3
#include "score.hip"
