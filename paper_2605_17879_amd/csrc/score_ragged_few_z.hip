// The scoring kernel for rank counts that fill no tiling exactly: up to 8 192 ranks, with the z output.
#define GD_SCORE_WANT_Z 1
#define GD_SCORE_RAGGED 1
#include "score.hip"
