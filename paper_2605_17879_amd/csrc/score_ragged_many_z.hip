// The scoring kernel for rank counts that fill no tiling exactly: more than 8 192 ranks, with the z output.
#define GD_SCORE_WANT_Z 1
#define GD_SCORE_RAGGED 2
#include "score.hip"
